"""GPU parity of the Ozaki-II (CRT) path against its CPU oracle, through the C
ABI. The integer conversion, the residues, the modular products and the CRT
rebuild are exact, and the rounding and alpha/beta are fixed by the model, so
the results must match bit for bit."""
import sys

import numpy as np
import pytest

from oracle import dd, metrics, ozaki2
from tests.gpu_util import bits_equal, dev, host, mismatch_report, require_gpu, torch
from workloads import kkr_operands, uniform_binade

import paper_2603_29975_amd as oz

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()
    yield
    torch.cuda.synchronize()


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _stored(X, trans):
    t = trans.upper()
    if t == "N":
        return X
    if t == "T":
        return np.ascontiguousarray(X.T)
    return np.ascontiguousarray(np.conj(X.T))


def _operands(kind, m, n, k, seed, nasty=False):
    A, B = uniform_binade(m, n, k, seed=seed, complex_=kind == "z")
    if nasty:
        rng = np.random.default_rng(seed + 1)
        A[rng.integers(0, m)] = 0.0                      # zero row
        B[:, rng.integers(0, n)] = 0.0                   # zero column
        A[rng.integers(0, m)] *= 2.0 ** -1060            # tiny row (subnormal entries)
        B[:, rng.integers(0, n)] *= 2.0 ** 900           # huge column
        A[rng.integers(0, m), rng.integers(0, k)] = 5e-324
    return A, B


def _run(kind, ta, tb, A, B, nmod, alpha=1.0, beta=0.0, C0=None):
    m, k = A.shape
    n = B.shape[1]
    Ad, lda = dev(_stored(A, ta))
    Bd, ldb = dev(_stored(B, tb))
    dt = np.complex128 if kind == "z" else np.float64
    if C0 is None:
        C0 = np.full((m, n), np.nan, dtype=dt)           # beta == 0 must not read C
    Cd, ldc = dev(C0.astype(dt))
    fn = oz.ozaki2_zgemm if kind == "z" else oz.ozaki2_dgemm
    rc = fn(ta, tb, m, n, k, alpha, Ad, lda, Bd, ldb, beta, Cd, ldc, nmod)
    assert rc == 0, oz.ozaki_status_string(rc)
    return host(Cd, m, n)


@pytest.mark.parametrize("kind", ["d", "z"])
@pytest.mark.parametrize("ta,tb,nmod", [("N", "N", 14), ("T", "N", 10), ("N", "C", 16),
                                        ("C", "T", 6), ("T", "T", 20), ("N", "N", 2)])
def test_ozaki2_bit_exact(kind, ta, tb, nmod):
    # several 64 x 64 residue tiles and 256-row rebuild blocks with ragged tails
    m, n, k = (300, 90, 140) if kind == "d" else (270, 70, 100)
    A, B = _operands(kind, m, n, k, seed=900 + nmod, nasty=True)
    _say("ozaki2", kind, ta, tb, nmod)
    got = _run(kind, ta, tb, A, B, nmod)
    ref = ozaki2.ozaki2_gemm("N", "N", A, B, nmod)
    assert bits_equal(got, ref), mismatch_report(got, ref)


@pytest.mark.parametrize("kind", ["d", "z"])
def test_ozaki2_alpha_beta_bit_exact(kind):
    m, n, k = 97, 130, 65
    A, B = _operands(kind, m, n, k, seed=910)
    rng = np.random.default_rng(911)
    C0 = rng.standard_normal((m, n))
    if kind == "z":
        C0 = C0 + 1j * rng.standard_normal((m, n))
        cases = [(0.5 - 1.25j, -2.0 + 0.5j), (1.0, 0.0), (1j, 1.0), (-0.3, 0.7j)]
    else:
        cases = [(0.5, -2.0), (1.0, 0.0), (-1.7, 1.0), (3.1, 0.25)]
    for alpha, beta in cases:
        _say("ozaki2 alpha/beta", kind, alpha, beta)
        got = _run(kind, "N", "N", A, B, 12, alpha, beta, C0 if beta != 0 else None)
        ref = ozaki2.ozaki2_gemm("N", "N", A, B, 12, alpha, beta, C0)
        assert bits_equal(got, ref), mismatch_report(got, ref)


@pytest.mark.parametrize("kind", ["d", "z"])
def test_ozaki2_quick_returns_nonfinite_and_tiny_shapes(kind):
    m, n, k = 33, 20, 17
    A, B = _operands(kind, m, n, k, seed=920)
    dt = np.complex128 if kind == "z" else np.float64
    C0 = (np.arange(m * n).reshape(m, n) + 0.5).astype(dt)
    got = _run(kind, "N", "N", A, B, 14, 0.0, 2.0, C0)
    assert bits_equal(got, ozaki2.ozaki2_gemm("N", "N", A, B, 14, 0.0, 2.0, C0))
    got = _run(kind, "N", "N", A[:, :0], B[:0, :], 14, 1.0, 3.0, C0)
    assert bits_equal(got, ozaki2.ozaki2_gemm("N", "N", A[:, :0], B[:0, :], 14, 1.0, 3.0, C0))
    A2, B2 = _operands(kind, 70, 90, 40, seed=921)
    A2[3, 7] = np.inf
    A2[60, 0] = np.nan
    B2[5, 80] = -np.inf
    got = _run(kind, "N", "N", A2, B2, 14)
    ref = ozaki2.ozaki2_gemm("N", "N", A2, B2, 14)
    assert bits_equal(got, ref), mismatch_report(got, ref)
    assert np.all(np.isnan(got[3])) and np.all(np.isnan(got[:, 80]))
    for (mm, nn, kk) in [(1, 1, 1), (1, 5, 3), (7, 1, 2), (3, 4, 1), (65, 257, 65)]:
        A3, B3 = _operands(kind, mm, nn, kk, seed=mm * 100 + nn * 10 + kk)
        got = _run(kind, "N", "N", A3, B3, 8)
        assert bits_equal(got, ozaki2.ozaki2_gemm("N", "N", A3, B3, 8)), (mm, nn, kk)


def test_ozaki2_integer_inputs_exact_and_accuracy_sweep():
    rng = np.random.default_rng(930)
    A = rng.integers(-1000, 1001, (70, 300)).astype(np.float64)
    B = rng.integers(-1000, 1001, (300, 50)).astype(np.float64)
    exact = (A.astype(np.int64) @ B.astype(np.int64)).astype(np.float64)
    assert np.array_equal(_run("d", "N", "N", A, B, 12), exact)
    # 160^3 DGEMM, entries u * 2^e, e in [-4, 4]: error falls with the moduli
    A, B = uniform_binade(160, 160, 160, seed=1001)
    hi, lo = dd.dd_gemm("N", "N", A, B)
    den = metrics.abs_product("N", "N", A, B)
    errs = {}
    for nmod in (8, 10, 12, 14, 16):
        got = _run("d", "N", "N", A, B, nmod)
        assert bits_equal(got, ozaki2.ozaki2_gemm("N", "N", A, B, nmod)), nmod
        errs[nmod] = metrics.err_comp(got, hi, lo, den)
    _say("ozaki2 err_comp", errs)
    assert all(errs[b] < errs[a] for a, b in ((8, 10), (10, 12), (12, 14), (14, 16)))
    assert errs[14] <= 1e-12


def test_ozaki2_kkr_2048_sampled_bit_exact_and_accuracy():
    # Full-size complex KKR workload (64 blocks of 32) at 14 moduli: the GPU
    # result equals the oracle on sampled rows/columns (the model is separable
    # by rows of op(A) and columns of op(B): exponents per row/column, beta
    # from N and K' only) and meets 1e-12 componentwise.
    A, B = kkr_operands(64, seed=1002)
    m = n = 2048
    got = _run("z", "N", "N", A, B, 14)
    rng = np.random.default_rng(78)
    rows = np.sort(rng.choice(m, 16, replace=False))
    cols = np.sort(rng.choice(n, 16, replace=False))
    ref = ozaki2.ozaki2_gemm("N", "N", A[rows], B[:, cols], 14)
    sub = got[np.ix_(rows, cols)]
    assert bits_equal(sub, ref), mismatch_report(sub, ref)
    ri, cj = np.meshgrid(rows, cols, indexing="ij")
    hi, lo = dd.dd_entries("N", "N", A, B, ri.ravel(), cj.ravel())
    den = metrics.denom_entries("N", "N", A, B, ri.ravel(), cj.ravel())
    err = metrics.err_comp(sub.ravel(), hi, lo, den)
    _say("kkr 2048 ozaki2 N=14 err_comp (sampled)", err)
    assert err <= 1e-12


def _planes(kind, m, n, k, nmod, ws_extra):
    """C of the same product with the library's workspace and with a caller's workspace of
    ozaki2_workspace_bytes + ws_extra."""
    A, B = _operands(kind, m, n, k, seed=970 + m + n, nasty=True)
    got = _run(kind, "N", "N", A, B, nmod)
    ws = torch.empty(oz.ozaki2_workspace_bytes(kind, m, n, k, nmod) + ws_extra, dtype=torch.uint8,
                     device="cuda")
    assert oz.ozaki_set_workspace(ws, ws.numel()) == 0
    try:
        other = _run(kind, "N", "N", A, B, nmod)
    finally:
        oz.ozaki_set_workspace(None, 0)
    return A, B, got, other


# (kind, m, n, k, moduli): tiles of 64 (one work item; ragged), of 128 (from 256 items) and of 256
# (from 192 items), row and column remainders on both sides of a tile, short and long contractions
@pytest.mark.parametrize("kind,m,n,k,nmod", [
    ("d", 1, 1, 1, 2), ("z", 63, 33, 70, 7), ("d", 65, 129, 300, 3), ("z", 257, 257, 33, 20),
    ("d", 511, 513, 129, 18), ("z", 513, 385, 64, 16), ("d", 1025, 1023, 260, 12)])
def test_ozaki2_residue_planes_and_fused_kernel_agree(kind, m, n, k, nmod):
    # a caller's workspace that ends with the residue planes takes the fused kernel, one with room
    # for a strip of 256 columns (the rest of C in further strips) and the library's own the planes
    A, B, got, fused = _planes(kind, m, n, k, nmod, 0)
    assert bits_equal(got, fused), mismatch_report(got, fused)
    strip = _planes(kind, m, n, k, nmod, nmod * 256 * ((m + 31) // 32 * 32))[3]
    assert bits_equal(got, strip), mismatch_report(got, strip)
    r, c = slice(max(0, m - 9), m), slice(max(0, n - 9), n)
    ref = ozaki2.ozaki2_gemm("N", "N", A[r], B[:, c], nmod)
    assert bits_equal(got[r, c], ref), mismatch_report(got[r, c], ref)


# Strips with enough products each for the residue planes (2.5e10): several of 1024 and 512
# columns, the last one ragged
@pytest.mark.parametrize("kind,m,n,k,nmod,columns", [("d", 1100, 2501, 2100, 14, 1024),
                                                     ("z", 1030, 650, 1500, 17, 512)])
def test_ozaki2_several_strips(kind, m, n, k, nmod, columns):
    A, B, got, strips = _planes(kind, m, n, k, nmod, nmod * columns * ((m + 31) // 32 * 32))
    assert bits_equal(got, strips), mismatch_report(got, strips)
    fused = _planes(kind, m, n, k, nmod, 0)[3]
    assert bits_equal(got, fused), mismatch_report(got, fused)
    c = np.r_[0:3, n // 2:n // 2 + 3, n - 3:n]
    ref = ozaki2.ozaki2_gemm("N", "N", A[-5:], B[:, c], nmod)
    assert bits_equal(got[-5:, c], ref), mismatch_report(got[-5:, c], ref)


@pytest.mark.parametrize("nmod", [14, 16, 17, 18, 20])
def test_ozaki2_rounding_at_ties(nmod):
    # sums 2^p (1 + 2^-53) and neighbours, alone and moved off the tie by a term 2^-q below: the
    # single rounding of the exact integer (limbs that cancel, ties to even, sticky tails)
    beta = oz.ozaki2_beta_bits(nmod, 4)
    rng = np.random.default_rng(nmod)
    m, n = 64, 48
    A = np.zeros((m, 4))
    B = np.zeros((4, n))
    half = beta // 2
    A[:, 0] = 1.0
    B[0] = 1.0 - 2.0 ** -rng.integers(1, half + 1, n)
    A[:, 1] = 2.0 ** -rng.integers(20, half + 1, m) * rng.choice([-1.0, 1.0], m)
    B[1] = 2.0 ** -rng.integers(20, 28, n)
    A[:, 2] = rng.choice([0.0, 1.0, -1.0], m) * 2.0 ** -beta
    B[2] = 2.0 ** -rng.integers(0, beta, n)
    A[:, 3] = rng.choice([0.0, -1.0], m)
    B[3] = B[0]
    got = _run("d", "N", "N", A, B, nmod)
    ref = ozaki2.ozaki2_gemm("N", "N", A, B, nmod)
    assert bits_equal(got, ref), mismatch_report(got, ref)


# Up to 128 packed contraction entries the residue kernel scans its rows itself: one entry, the
# limit and one past it, in every storage order, with Inf and NaN, for both digit forms (20 moduli
# take the unsigned one)
@pytest.mark.parametrize("nmod", [9, 20])
@pytest.mark.parametrize("kind,m,n,k", [("d", 65, 17, 1), ("d", 33, 130, 128), ("d", 33, 130, 129),
                                        ("z", 66, 31, 64), ("z", 66, 31, 65), ("z", 1, 1, 40)])
def test_ozaki2_short_contractions(nmod, kind, m, n, k):
    for ta, tb in (("N", "N"), ("T", "N"), ("N", "T"), ("C", "C")):
        for bad in (False, True):
            A, B = _operands(kind, m, n, k, seed=990 + k, nasty=m > 1)
            if bad:
                A[m // 2, k - 1], B[0, n // 2] = np.nan, -np.inf
            _say("ozaki2 short", kind, (m, n, k), nmod, ta, tb, bad)
            got = _run(kind, ta, tb, A, B, nmod)
            ref = ozaki2.ozaki2_gemm("N", "N", A, B, nmod)
            assert bits_equal(got, ref), mismatch_report(got, ref)


# More groups of four columns than a grid has blocks along y (65535), in one strip
@pytest.mark.parametrize("kind,m,n,k,nmod", [("d", 32, 262149, 8, 8), ("z", 17, 131075, 5, 16)])
def test_ozaki2_wide_products(kind, m, n, k, nmod):
    A, B = _operands(kind, m, n, k, seed=995)
    _say("ozaki2 wide", kind, (m, n, k), nmod)
    got = _run(kind, "N", "N", A, B, nmod)
    cols = np.concatenate([np.arange(40), np.arange(n // 2, n // 2 + 9), np.arange(n - 40, n),
                           np.random.default_rng(996).choice(n, 200, replace=False)])
    ref = ozaki2.ozaki2_gemm("N", "N", A, B[:, cols], nmod)
    assert bits_equal(got[:, cols], ref), mismatch_report(got[:, cols], ref)
    assert np.all(np.isfinite(got.view(np.float64)))


def test_ozaki2_residue_bytes_beside_the_workspace():
    # a workspace that a real product left, with room for the residue planes but not for the
    # products' residue bytes behind them, gives the bits of one that grew for the call
    m = n = k = 2048
    A, B = kkr_operands(64, seed=1002)
    assert oz.ozaki_finalize() == 0
    ref = _run("z", "N", "N", A, B, 14)
    assert oz.ozaki_finalize() == 0
    X = torch.zeros((4096, 4096), dtype=torch.float64, device="cuda")
    assert oz.ozaki_dgemm("N", "N", 3072, 4096, 4096, 1.0, X, 3072, X, 4096, 0.0, torch.empty_like(X), 3072, 12) == 0
    need = oz.ozaki2_workspace_bytes("z", m, n, k, 14)
    assert need <= oz.ozaki_workspace_bytes("d", 3072, 4096, 4096, 12) < need + 14 * m * 2 * n
    for _ in range(2):
        _say("ozaki2 beside the workspace")
        got = _run("z", "N", "N", A, B, 14)
        assert bits_equal(got, ref), mismatch_report(got, ref)
    assert oz.ozaki_finalize() == 0


# Wide products on both sides of 64 rows, where the fused kernel gives way to residue bytes
@pytest.mark.parametrize("nmod", [14, 19])
@pytest.mark.parametrize("kind,m,n,k", [("d", 1, 32700, 70), ("d", 64, 32765, 33), ("z", 64, 16383, 20),
                                        ("d", 65, 32765, 33)])
def test_ozaki2_thin_products(nmod, kind, m, n, k):
    A, B = _operands(kind, m, n, k, seed=1010 + m, nasty=m > 1)
    _say("ozaki2 thin", kind, (m, n, k), nmod)
    got = _run(kind, "N", "N", A, B, nmod)
    cols = np.unique(np.concatenate([np.arange(70), np.arange(n - 70, n),
                                     np.random.default_rng(1011).choice(n, 100, replace=False)]))
    ref = ozaki2.ozaki2_gemm("N", "N", A, B[:, cols], nmod)
    assert bits_equal(got[:, cols], ref), mismatch_report(got[:, cols], ref)
