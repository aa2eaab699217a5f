"""Performance cases of the library: the calls a solver makes, through the public entry points.

``listed()`` gives the fixed cases, ``draw(rng)`` another one of the same ranges. ``prepare``
draws the operands from a seed, ``run`` makes one call, ``work`` counts the bytes and operations
the call cannot do without (INT8 operations for the emulated products: the slice pairs or moduli
the caller asked for), ``exact`` gives the same result in plain 64-bit arithmetic.

The shipped tuning table is loaded as bench.py loads it. Matrices are column-major device
buffers, held as torch tensors of shape (columns, leading dimension).
"""
import math
import os

import numpy as np
import torch

import paper_2603_29975_amd as oz
from paper_2603_29975_amd import blas, selector

PKG = os.path.dirname(os.path.abspath(oz.__file__))
Z, D = torch.complex128, torch.float64


def listed():
    return [
        # one 32 x 32 site block of a KKR matrix times another, through the tensor convenience:
        # the smallest call, where launches and latency count
        _gemm("z_block32", "z", 32, 32, 32, 7, family="gauss", entry="matmul"),
        # the smallest benchmark product: real, entries over eight binades
        _gemm("d_256", "d", 256, 256, 256, 7, family="binade"),
        # an ordinary BLAS call: odd sizes, padded leading dimensions, C^H and T, alpha and beta
        _gemm("z_ragged", "z", 517, 389, 1031, 8, ta="C", tb="T", family="scaled", pad=3, ab=True),
        # a large real product with seven-bit slices
        _gemm("d_4096", "d", 4096, 4096, 4096, 7, ta="N", tb="T", family="binade"),
        # the KKR product of the benchmark: I - T G times a Gaussian block, eight-bit slices
        _gemm("z_kkr2048", "z", 2048, 2048, 2048, 6, split="b8", family="kkr"),
        # the benchmark's headline: rows and columns scaled over 60 binades
        _gemm("z_ill16384", "z", 16384, 16384, 16384, 6, split="b8", family="scaled"),
        # 512 uneven block products of one inversion step at a fixed slice count
        {"name": "z_batched512", "kind": "batched", "count": 512, "s": 7, "sizes": 1003, "odd": False},
        # the same batch with the learned slice counts and the residual probe
        {"name": "z_auto512", "kind": "batched", "count": 512, "s": 0, "sizes": 1003, "odd": False},
        # the KKR product by residues, at one of the paper's moduli counts
        _gemm("z_crt2048", "z", 2048, 2048, 2048, 0, moduli=14, family="kkr"),
        # the step around the products: LU and inverse of a KKR matrix
        {"name": "z_inverse2048", "kind": "lu", "n": 2048, "nb": 128, "s": 6, "split": "b8"},
        # one training step of the slice selector (forward, loss and gradient) at its batch size
        {"name": "mlp_step256", "kind": "mlp", "batch": 256},
        # the paper's use: a host program's ZGEMM, intercepted; the copies are part of the call
        {"name": "z_host2048", "kind": "host", "m": 2048, "n": 2048, "k": 2048, "s": 7},
    ]


def _gemm(name, dtype, m, n, k, s, split="t7", ta="N", tb="N", family="gauss", pad=0, ab=False,
          entry="blas", moduli=0):
    c = {"name": name, "kind": "gemm", "dtype": dtype, "ta": ta, "tb": tb, "m": m, "n": n, "k": k,
         "s": s, "split": split, "family": family, "pad": pad, "ab": ab, "entry": entry,
         "moduli": moduli}
    if not name:
        del c["name"]
    return c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemm"] * 6 + ["crt"] * 2 + ["batched", "auto", "lu", "mlp", "host"])
    if kind in ("gemm", "crt"):
        m, n, k = (_log(rng, 16, 8192) for _ in range(3))
        dtype = rng.choice("zzd")
        t = {"z": "NTC", "d": "NT"}[dtype]
        split = rng.choice(["t7", "b8"]) if kind == "gemm" else "t7"
        s = rng.randint(4, 8 if split == "b8" else 10) if kind == "gemm" else 0
        return _gemm("", dtype, m, n, k, s, split, rng.choice(t), rng.choice(t),
                     rng.choice(["gauss", "scaled", "binade"]), rng.choice([0, 0, 1, 8]),
                     rng.random() < 0.5, moduli=rng.randint(8, 18) if kind == "crt" else 0)
    if kind in ("batched", "auto"):
        return {"kind": "batched", "count": _log(rng, 8, 512), "s": rng.randint(5, 9) if kind == "batched" else 0,
                "sizes": rng.randint(1, 10 ** 6), "odd": rng.random() < 0.5}
    if kind == "lu":
        split = rng.choice(["t7", "b8"])
        return {"kind": "lu", "n": _log(rng, 64, 3000), "nb": rng.choice([32, 64, 96, 128]),
                "s": rng.choice([0, 5, 6, 7]), "split": split}
    if kind == "mlp":
        return {"kind": "mlp", "batch": _log(rng, 16, 8192)}
    m, n, k = (_log(rng, 64, 3000) for _ in range(3))
    return {"kind": "host", "m": m, "n": n, "k": k, "s": rng.randint(5, 8)}


# ------------------------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=dtype)


def _power(g, shape, lo, hi):
    """2^r with r a uniform integer in [lo, hi]."""
    return torch.ldexp(torch.ones(shape, device="cuda", dtype=D),
                       torch.randint(lo, hi + 1, shape, generator=g, device="cuda"))


def _operand(g, rows, cols, dtype, family, scale_rows):
    """The rows x cols matrix op(A) or op(B) of one family."""
    if family == "binade":  # entries u 2^e, e in [-4, 4]
        def part():
            u = torch.rand((rows, cols), generator=g, device="cuda", dtype=D) * 2 - 1
            return u * _power(g, (rows, cols), -4, 4)
        return torch.complex(part(), part()) if dtype is Z else part()
    if family == "kkr" and scale_rows:  # I - T G: T block diagonal, G decaying with block distance
        nb = -(-rows // 32)
        mag = 10.0 ** (-3 * torch.rand((nb, 32, 32), generator=g, device="cuda", dtype=D))
        T = torch.polar(mag, 2 * math.pi * torch.rand((nb, 32, 32), generator=g, device="cuda", dtype=D))
        bi, bj = torch.arange(nb * 32, device="cuda") // 32, torch.arange(cols, device="cuda") // 32
        G = _normal(g, (nb * 32, cols), Z) / (1.0 + (bi[:, None] - bj[None, :]).abs())
        X = -torch.bmm(T, G.view(nb, 32, cols)).view(nb * 32, cols)[:rows]
        X.diagonal().add_(1.0)
        return X.contiguous()
    X = _normal(g, (rows, cols), dtype)
    if family == "scaled":  # rows of A, columns of B times 2^r, r in [-30, 30]
        X *= _power(g, (rows, 1) if scale_rows else (1, cols), -30, 30)
    return X


def _stored(X, trans, ld_pad):
    """Column-major storage (columns, ld) of the matrix whose op() is X."""
    if trans == "C":
        X = X.conj()
    rows, cols = X.shape if trans == "N" else X.shape[::-1]
    S = torch.zeros((cols, rows + ld_pad), dtype=X.dtype, device="cuda")
    S[:, :rows] = X.T if trans == "N" else X
    return S


def _gemm_inputs(c, seed):
    g = _gen(seed)
    dt = Z if c["dtype"] == "z" else D
    A = _operand(g, c["m"], c["k"], dt, c["family"], True)
    B = _operand(g, c["k"], c["n"], dt, c["family"], False)
    C = _normal(g, (c["n"], c["m"] + c["pad"]), dt) if c["ab"] else None
    return A, B, C


def _scalars(c):
    if not c["ab"]:
        return 1.0, 0.0
    return (0.75 - 0.5j, -0.25 + 1.0j) if c["dtype"] == "z" else (-0.75, 0.5)


def _sizes(c):
    """m, n, k per problem: 32 j with P(j) ~ 1/j, j <= 32; `odd` takes up to 31 off each."""
    rng = np.random.default_rng(c["sizes"])
    j = np.arange(1, 33)
    d = rng.choice(j, size=(c["count"], 3), p=(1.0 / j) / np.sum(1.0 / j)) * 32
    if c["odd"]:
        d = d - rng.integers(0, 32, size=d.shape)
    return [[int(x) for x in row] for row in d]


def _batched_inputs(c, seed):
    """Gaussian entries times 2^-floor(sigma u), rows (columns) times 2^r, sigma ~ U[0, 20] per
    matrix; column-major, in one buffer per operand."""
    g, rng = _gen(seed), np.random.default_rng(seed)
    A, B = [], []
    for m, n, k in _sizes(c):
        for out, rows, cols, side in ((A, m, k, 1), (B, k, n, 0)):
            sg = rng.uniform(0.0, 20.0)
            X = _normal(g, (cols, rows), Z)
            u = torch.rand((cols, rows), generator=g, device="cuda", dtype=D)
            r = torch.randint(0, int(sg) + 1, (1, rows) if side else (cols, 1), generator=g, device="cuda")
            out.append(X * torch.ldexp(torch.ones((), device="cuda", dtype=D), r - torch.floor(sg * u).long()))
    return A, B


def _mlp_inputs(c, seed):
    """Feature-like rows (fractions that sum to one per operand side), targets 3..12, weights of
    the usual He scale with small biases."""
    g, b = _gen(seed), c["batch"]
    f = torch.rand((b, 63), generator=g, device="cuda") ** 6
    X = torch.cat([f[:, :32] / f[:, :32].sum(1, keepdim=True), f[:, 32:] / f[:, 32:].sum(1, keepdim=True),
                   torch.rand((b, 1), generator=g, device="cuda")], 1).contiguous()
    t = torch.randint(3, 13, (b,), generator=g, device="cuda").float()
    w = torch.randn(oz.MLP_PARAMS, generator=g, device="cuda")
    for o, n, fan in ((0, 8192, 64), (8192, 128, 0), (8320, 16384, 128), (24704, 128, 0), (24832, 128, 128), (24960, 1, 0)):
        w[o:o + n] *= math.sqrt(2.0 / fan) if fan else 0.1
    return X, t, w


# ------------------------------------------------------------------------------------ cases
def _ok(rc, what):
    if rc != 0:
        raise oz.OzakiError(rc, what)


def prepare(case, seed):
    oz.ozaki_tune_clear()
    _ok(oz.ozaki_tune_load(os.path.join(PKG, "tune_gfx950.json")), "tune_load")
    c, kind = case, case["kind"]
    if kind == "gemm":
        A, B, C0 = _gemm_inputs(c, seed)
        if c["entry"] == "matmul":
            return {"case": c, "A": A.contiguous(), "B": B.contiguous()}
        dt = A.dtype
        A, B = _stored(A, c["ta"], c["pad"]), _stored(B, c["tb"], c["pad"])
        C = torch.zeros((c["n"], c["m"] + c["pad"]), dtype=dt, device="cuda") if C0 is None else C0.clone()
        return {"case": c, "A": A, "B": B, "C": C, "C0": C0}
    if kind == "batched":
        A, B = _batched_inputs(c, seed)
        mnk = _sizes(c)
        flat = torch.zeros(sum(m * n for m, n, _ in mnk), dtype=Z, device="cuda")
        C, at = [], 0
        for m, n, _ in mnk:
            C.append(flat[at:at + m * n])
            at += m * n
        m, n, k = ([d[i] for d in mnk] for i in range(3))
        if c["s"] == 0:
            theta, margin, target, meta = selector.load(os.path.join(PKG, "selector_weights.npz"), with_meta=True)
            _ok(oz.ozaki_load_selector(theta, margin, target, float(meta["kappa"])), "load_selector")
        nb = c["count"]
        return {"case": c, "A": A, "B": B, "C": C, "flat": flat, "m": m, "n": n, "k": k,
                "N": ["N"] * nb, "one": [1.0] * nb, "zero": [0.0] * nb,
                "s": [c["s"]] * nb if c["s"] else None}
    if kind == "lu":
        n = c["n"]
        A = _operand(_gen(seed), n, n, Z, "kkr", True).T.contiguous()
        return {"case": c, "A": A, "LU": torch.empty_like(A), "X": torch.empty_like(A),
                "ipiv": torch.zeros(n, dtype=torch.int64, device="cuda")}
    if kind == "mlp":
        X, t, w = _mlp_inputs(c, seed)
        b = c["batch"]
        state = torch.zeros(oz.ozaki_mlp_state_bytes() // 4 + 16, dtype=torch.float32, device="cuda")
        state[:oz.MLP_PARAMS] = w
        _ok(oz.ozaki_mlp_refresh(state), "mlp_refresh")
        return {"case": c, "X": X, "t": t, "state": state,
                "scratch": torch.zeros(oz.ozaki_mlp_scratch_bytes(b) // 4 + 64, dtype=torch.float32, device="cuda"),
                "y": torch.zeros(b, dtype=torch.float32, device="cuda"),
                "loss": torch.zeros(1, dtype=torch.float32, device="cuda")}
    A, B, _ = _gemm_inputs({**c, "dtype": "z", "family": "kkr", "ab": False}, seed)
    _ok(blas.ozaki_blas_config(slices=c["s"]), "blas_config")
    return {"case": c, "A": A.T.contiguous().cpu().numpy(), "B": B.T.contiguous().cpu().numpy(),
            "C": np.zeros((c["n"], c["m"]), dtype=np.complex128)}


def run(state):
    st, c = state, state["case"]
    kind = c["kind"]
    if kind == "gemm":
        if c["entry"] == "matmul":
            oz.ozaki_set_split(c["split"])
            return oz.matmul(st["A"], st["B"], slices=c["s"])
        A, B, C = st["A"], st["B"], st["C"]
        if st["C0"] is not None:  # the caller's C, which the product is added to
            C.copy_(st["C0"])
        al, be = _scalars(c)
        args = (c["ta"], c["tb"], c["m"], c["n"], c["k"], al, A, A.shape[1], B, B.shape[1], be, C, C.shape[1])
        if c["moduli"]:
            _ok((oz.ozaki2_zgemm if c["dtype"] == "z" else oz.ozaki2_dgemm)(*args, c["moduli"]), "ozaki2")
        else:
            oz.ozaki_set_split(c["split"])
            _ok((oz.ozaki_zgemm if c["dtype"] == "z" else oz.ozaki_dgemm)(*args, c["s"]), "ozaki")
        return C
    if kind == "batched":
        used = []
        _ok(oz.ozaki_zgemm_batched(st["N"], st["N"], st["m"], st["n"], st["k"], st["one"], st["A"], st["m"],
                                   st["B"], st["k"], st["zero"], st["C"], st["m"], c["count"], st["s"], used),
            "batched")
        return {"C": st["flat"], "slices": np.array(used, dtype=np.int64)}
    if kind == "lu":
        n = c["n"]
        oz.ozaki_set_split(c["split"])
        st["LU"].copy_(st["A"])  # the solver assembles its matrix there; factored in place
        _ok(oz.ozaki_zgetrf(n, st["LU"], n, st["ipiv"], c["nb"], c["s"]), "zgetrf")
        _ok(oz.ozaki_zgetri(n, st["LU"], n, st["ipiv"], st["X"], n, c["nb"], c["s"]), "zgetri")
        return {"LU": st["LU"], "X": st["X"], "ipiv": st["ipiv"]}
    if kind == "mlp":
        b = c["batch"]
        _ok(oz.ozaki_mlp_forward(st["state"], b, st["X"], st["y"], st["scratch"]), "mlp_forward")
        _ok(oz.ozaki_mlp_backward(st["state"], b, st["y"], st["t"], 4.0, st["loss"], st["scratch"]), "mlp_backward")
        return {"y": st["y"], "loss": st["loss"], "grad": st["state"][3 * oz.MLP_PARAMS:4 * oz.MLP_PARAMS]}
    oz.ozaki_set_split("t7")
    blas.zgemm_("N", "N", c["m"], c["n"], c["k"], 1.0, st["A"], c["m"], st["B"], c["k"], 0.0, st["C"], c["m"])
    return st["C"]


def work(case):
    c, kind = case, case["kind"]
    if kind in ("gemm", "host"):
        z = kind == "host" or c["dtype"] == "z"
        m, n, k = c["m"], c["n"], c["k"]
        times = c.get("moduli") or c["s"] * (c["s"] + 1) // 2
        return {"bytes": (16 if z else 8) * (m * k + k * n + (2 if c.get("ab") else 1) * m * n),
                "flops": times * (8 if z else 2) * m * n * k}
    if kind == "batched":
        pairs = (c["s"] or 7) * ((c["s"] or 7) + 1) // 2
        return {"bytes": sum(16 * (m * k + k * n + m * n) for m, n, k in _sizes(c)),
                "flops": sum(pairs * 8 * m * n * k for m, n, k in _sizes(c))}
    if kind == "lu":
        n = c["n"]
        return {"bytes": 16 * 3 * n * n + 8 * n, "flops": max(1, c["s"] * (c["s"] + 1) // 2) * 8 * n ** 3}
    b = c["batch"]
    return {"bytes": 4 * (b * 66 + 2 * oz.MLP_PARAMS), "flops": 6 * b * (64 * 128 + 128 * 128 + 128)}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("gemm", "host"):
        host = kind == "host"
        A, B, C = _gemm_inputs({**c, "dtype": "z", "family": "kkr", "ab": False} if host else c, seed)
        if host:
            return (A @ B).T.contiguous().cpu().numpy()
        P = A @ B
        if c["entry"] == "matmul":
            return P
        al, be = _scalars(c)
        if C is None:
            C = torch.zeros((c["n"], c["m"] + c["pad"]), dtype=P.dtype, device="cuda")
        V = C[:, :c["m"]]
        V.copy_(al * P.T + be * V if c["ab"] else P.T)
        return C
    if kind == "batched":
        A, B = _batched_inputs(c, seed)
        return {"C": torch.cat([(b @ a).reshape(-1) for a, b in zip(A, B)]), "slices": None}
    if kind == "lu":
        A = _operand(_gen(seed), c["n"], c["n"], Z, "kkr", True).cpu()
        return {"LU": None, "X": torch.linalg.inv(A).T.contiguous(), "ipiv": None}
    X, t, w = (v.double() for v in _mlp_inputs(c, seed))
    w.requires_grad_(True)
    h = torch.relu(X @ w[:8192].view(128, 64).T + w[8192:8320])
    h = torch.relu(h @ w[8320:24704].view(128, 128).T + w[24704:24832])
    y = h @ w[24832:24960] + w[24960]
    loss = (torch.where(y < t, 4.0, 1.0) * (y - t) ** 2).mean()
    grad, = torch.autograd.grad(loss, w)
    return {"y": y.detach(), "loss": loss.detach().reshape(1), "grad": grad}
