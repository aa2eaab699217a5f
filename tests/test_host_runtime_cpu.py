"""Host runtime of libozaki and its BLAS interposer without a GPU: child processes load
fake_hip.cpp (device memory as a budget, kernels and copies recorded) in front of the HIP
runtime, make library calls and print what these asked of it."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_PRELUDE = r"""
import ctypes, sys
sys.path.insert(0, %(root)r)
fake = ctypes.CDLL(%(fake)r, mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
fake.fake_used.restype = ctypes.c_size_t
fake.fake_pinned.restype = ctypes.c_void_p
fake.fake_pinned.argtypes = fake.fake_budget.argtypes = [ctypes.c_size_t]
import paper_2603_29975_amd as oz
lib = oz.library()
P = 1 << 40                                   # operands: addresses that no kernel reads
MIB = 1 << 20

def log():
    return [l.split() for l in fake.fake_log().decode().splitlines()]

def of(lines, *what):
    return [l for l in lines if l[0] in what]

def dgemm(m, n, k, s=7):
    return lib.ozaki_dgemm(b"N", b"N", m, n, k, 1.0, P, m, P, k, 0.0, P, m, s)

def crt(kind, m, n, k, moduli):
    one, zero = (1.0, 0.0) if kind == "d" else (oz.ozaki_z(1.0, 0.0), oz.ozaki_z(0.0, 0.0))
    f = lib.ozaki2_dgemm if kind == "d" else lib.ozaki2_zgemm
    return f(b"N", b"N", m, n, k, one, P, m, P, k, zero, P, m, moduli)

def need2(kind, m, n, k, moduli):
    return lib.ozaki2_workspace_bytes(kind.encode(), m, n, k, moduli)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", out],
                   check=True, timeout=300)
    return out


@pytest.fixture
def child(fake):
    def run(script):
        r = subprocess.run([sys.executable, "-c", _PRELUDE % {"root": ROOT, "fake": fake} + script],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.returncode, r.stdout, r.stderr)
    return run


def test_workspace_moves_only_for_a_call_that_does_not_fit(child):
    # 2048^3 complex at 14 moduli: 352 MiB of residue planes and 112 MiB for the products' residue
    # bytes; a buffer in between holds the call, so its address, which captured graphs keep, stays
    child(r"""
case = ("z", 2048, 2048, 2048, 14)
need = need2(*case)
assert dgemm(3072, 4096, 4096, 12) == 0       # needs a little more
made = of(log(), "malloc")
assert len(made) == 1 and need < int(made[0][1]) < need + 32 * MIB, (need, made)
for call in range(3):
    assert crt(*case) == 0
    made = log()
    assert not of(made, "free", "nomem")
    # the residue bytes go to 256 MiB of their own, asked for once
    assert of(made, "malloc") == ([["malloc", str(256 * MIB)]] if call == 0 else [])
    assert any("k_oz2mod" in l[1] for l in of(made, "launch"))
assert lib.ozaki_finalize() == 0 and fake.fake_used() == 0
print("ok")
""")


def test_workspace_of_a_first_ozaki2_call_holds_the_residue_bytes(child):
    child(r"""
case = ("z", 2048, 2048, 2048, 14)
assert crt(*case) == 0
made = log()
assert int(of(made, "malloc")[0][1]) >= need2(*case) + 14 * 2048 * 4096
assert any("k_oz2mod" in l[1] for l in of(made, "launch"))
for _ in range(2):
    assert crt(*case) == 0
    assert not of(log(), "malloc", "free")
print("ok")
""")


def test_workspace_without_room_for_the_residue_bytes_is_asked_for_once(child):
    child(r"""
case = ("z", 2048, 2048, 2048, 14)
fake.fake_budget(need2(*case) + MIB)
assert crt(*case) == 0
made = log()
assert len(of(made, "malloc")) == 1 and any("k_oz2gemm" in l[1] for l in of(made, "launch"))
for _ in range(3):
    assert crt(*case) == 0
    assert not of(log(), "malloc", "free", "nomem")
print("ok")
""")


def test_capture_allocates_no_optional_space(child):
    child(r"""
case = ("z", 2048, 2048, 2048, 14)
fake.fake_capture(1)
assert crt(*case) == 0
made = of(log(), "malloc")
assert len(made) == 1 and int(made[0][1]) == need2(*case), made
fake.fake_capture(0)
assert crt(*case) == 0 and len(of(log(), "malloc")) == 1
print("ok")
""")


@pytest.mark.parametrize("mib", [100, 20])
def test_small_product_on_a_nearly_full_device(child, mib):
    # less free memory than the buffer's usual first size
    child(r"""
fake.fake_budget(%d * MIB)
assert dgemm(64, 64, 64) == 0
assert crt("z", 64, 64, 64, 14) == 0
log()
assert dgemm(64, 64, 64) == 0
assert not of(log(), "malloc", "free", "nomem")
fake.fake_budget(0)
assert dgemm(4096, 4096, 4096) == 2           # OZAKI_ERR_ALLOC
print("ok")
""" % mib)


@pytest.mark.parametrize("kind,m,n,moduli", [("d", 32, 262145, 8), ("d", 1, 2000000, 2), ("z", 16, 131073, 16),
                                             ("z", 300, 200000, 3), ("d", 500000, 700000, 2)])
def test_wide_ozaki2_products_stay_within_the_grid_limits(child, kind, m, n, moduli):
    # in the library's own workspace, and in one that holds the residue bytes of every column
    child(r"""
case = (%r, %d, %d, 8, %d)
fake.fake_budget(1 << 46)
for ws in (0, need2(*case) + (1 << 43)):
    assert lib.ozaki_set_workspace(P if ws else None, ws) == 0
    assert crt(*case) == 0, fake.fake_log()
    made = log()
    assert of(made, "launch") and not of(made, "refused")
    assert any("k_oz2rebuild" in l[1] for l in made)
print("ok")
""" % (kind, m, n, moduli))


# strips: how many the two-kernel path is cut into, 0 for the fused kernel
@pytest.mark.parametrize("kind,m,n,k,moduli,columns,strips", [
    ("z", 64, 4096, 64, 14, 256, 0),          # many small strips: the fused kernel is faster
    ("d", 100, 8000, 100, 8, 1024, 0),
    ("z", 512, 4096, 512, 18, 1024, 0),
    ("d", 4096, 4096, 4096, 8, 256, 16),      # strips that fill the chip for long enough
    ("d", 1100, 2501, 2100, 14, 1024, 3),
    ("z", 1030, 650, 1500, 17, 512, 3),
    ("z", 2048, 2048, 2048, 14, 1024, 4),
    ("z", 64, 4096, 64, 14, 8192, 1)])        # every column at once
def test_ozaki2_strips_in_a_limited_workspace(child, kind, m, n, k, moduli, columns, strips):
    child(r"""
case = (%r, %d, %d, %d, %d)
ws = need2(*case) + case[4] * %d * ((case[1] + 31) // 32 * 32)
assert lib.ozaki_set_workspace(P, ws) == 0
assert crt(*case) == 0
names = [l[1] for l in of(log(), "launch")]
assert sum("k_oz2mod" in x for x in names) == %d, names
assert sum("k_oz2gemm" in x for x in names) == %d, names
print("ok")
""" % (kind, m, n, k, moduli, columns, strips, strips == 0))


_BLAS = r"""
from paper_2603_29975_amd import blas
import numpy as np
b = blas.library()
def zgemm(n, A, ld, B, C):
    i, z = (lambda v: ctypes.byref(ctypes.c_int(v))), (lambda v: ctypes.byref(oz.ozaki_z(v, 0.0)))
    b.zgemm_(b"N", b"N", i(n), i(n), i(n), z(1.0), A, i(ld), B, i(ld), z(0.0), C, i(ld))
def copies():
    return [l for l in log() if l[0] in ("copy", "copy2d", "copyasync", "pinned")]
"""


def test_interposer_takes_memory_known_to_the_runtime_straight_over_the_link(child):
    # 1000 x 1000 complex (16 MB): pinned arrays in one copy each, packed or pitched, no staging;
    # device memory, which the host may not touch (here: not at all), the same way
    child(_BLAS + r"""
n, size = 1000, 16 * 1000 * 1000
pinned = [fake.fake_pinned(size + 16 * 1000 * 8) for _ in range(3)]
device = []
for _ in range(3):
    p = ctypes.c_void_p()
    assert fake.hipMalloc(ctypes.byref(p), ctypes.c_size_t(size + 16 * 1000 * 8)) == 0
    device.append(p.value)
for A, B, C in (pinned, device, [x + 16 for x in pinned]):
    log()
    zgemm(n, A, n, B, C)
    assert copies() == [["copy", str(size), "1"]] * 2 + [["copy", str(size), "2"]]
    zgemm(n, A, n + 8, B, C)
    assert copies() == [["copy2d", str(16 * n), str(n), "1"]] * 2 + [["copy2d", str(16 * n), str(n), "2"]]
print("ok")
""")


def test_interposer_stages_large_or_pitched_pageable_arrays(child):
    child(_BLAS + r"""
def arrays(n, ld):
    return [np.zeros((n, ld), dtype=np.complex128) for _ in range(3)]
for n, ld, staged in ((1000, 1000, True), (100, 100, False), (100, 101, True)):
    X = arrays(n, ld)
    log()
    zgemm(n, X[0].ctypes.data, ld, X[1].ctypes.data, X[2].ctypes.data)
    got = {l[0] for l in copies()}
    assert ("copyasync" in got) == staged and ("copy" in got) != staged and "copy2d" not in got, (n, ld, got)
print("ok")
""")


# One scan-and-split kernel for operands up to so many blocks, by the packed contraction (k, or 2k
# complex, up to 64, 128, 256, 512); beyond, a scan and a split of both operands
@pytest.mark.parametrize("kind,m,n,k,fused", [
    ("d", 64, 500000, 64, True), ("z", 64, 500000, 32, True),
    ("d", 64, 100000, 128, True), ("z", 64, 30000, 64, True), ("z", 64, 100000, 64, False),
    ("z", 100000, 64, 64, False),
    ("d", 8000, 64, 192, True), ("d", 30000, 64, 192, False), ("z", 64, 8000, 96, True),
    ("d", 2000, 2000, 256, True), ("d", 64, 30000, 256, False), ("z", 64, 100000, 128, False),
    ("d", 512, 512, 512, True), ("z", 1200, 1200, 256, False), ("d", 64, 64, 513, False)])
def test_scan_and_split_kernels_by_size(child, kind, m, n, k, fused):
    child(r"""
kind, m, n, k, fused = %r, %d, %d, %d, %r
assert dgemm(m, n, k) == 0 if kind == "d" else lib.ozaki_zgemm(
    b"N", b"N", m, n, k, oz.ozaki_z(1.0, 0.0), P, m, P, k, oz.ozaki_z(0.0, 0.0), P, m, 7) == 0
names = [l[1] for l in of(log(), "launch")]
assert any("k_prep" in x for x in names) == fused, names
assert any("k_scan" in x for x in names) != fused and any("k_split" in x for x in names) != fused, names
print("ok")
""" % (kind, m, n, k, fused))


# k_ozgemm<S, WJ, WI, IB, ...> of a product without a table entry: 64 x 64 tiles are <S, 4, 1, 4>,
# 128 x 64 ones <S, 8, 1, 4>
@pytest.mark.parametrize("m,n,k,s,tile", [(64, 100000, 128, 6, "4ELi1ELi4"), (16, 40000, 700, 5, "4ELi1ELi4"),
                                          (64, 100000, 128, 7, "8ELi1ELi4"), (65, 100000, 128, 7, "8ELi1ELi4")])
def test_tiles_of_thin_products(child, m, n, k, s, tile):
    child(r"""
m, n, k, s = %d, %d, %d, %d
assert lib.ozaki_zgemm(b"N", b"N", m, n, k, oz.ozaki_z(1.0, 0.0), P, m, P, k, oz.ozaki_z(0.0, 0.0), P, m, s) == 0
names = [l[1] for l in of(log(), "launch")]
assert any("k_ozgemmILi%%dELi%s" %% s in x for x in names), names
print("ok")
""" % (m, n, k, s, tile))


# The kernel of the modular products: k_oz2gemm (fused), or k_oz2mod by its tile, <2, 4, 8, 4> 256 x
# 256, <2, 2, 4, 4> 128 x 128, <2, 2, 2, 2> 64 x 64
@pytest.mark.parametrize("kind,m,n,k,moduli,kernel", [
    ("z", 16, 40000, 16, 8, "k_oz2modILi2ELi2ELi2E"), ("z", 100, 40000, 16, 14, "k_oz2modILi2ELi2ELi4E"),
    ("z", 40000, 8, 100, 14, "k_oz2modILi2ELi2ELi2E"), ("z", 200, 40000, 16, 14, "k_oz2modILi2ELi4ELi8E"),
    ("z", 64, 16000, 700, 14, "k_oz2gemm"), ("z", 65, 16000, 700, 14, "k_oz2mod"),
    ("z", 64, 25000, 16, 14, "k_oz2mod"), ("z", 64, 40000, 100, 13, "k_oz2mod"),
    ("d", 64, 200000, 200, 18, "k_oz2gemm")])
def test_ozaki2_kernels_of_thin_products(child, kind, m, n, k, moduli, kernel):
    child(r"""
assert crt(%r, %d, %d, %d, %d) == 0
names = [l[1] for l in of(log(), "launch")]
assert any("%s" in x for x in names), names
print("ok")
""" % (kind, m, n, k, moduli, kernel))


# The grouped GEMM of a batch, k_ozgemm<S, WJ, WI, IB, ...>: the sizes of test_gpu_batched.py and the
# shapes that they are there for
@pytest.mark.parametrize("s,sizes,tile", [
    (6, [(500, 500, 70)] * 24, "8ELi1ELi8"), (7, [(500, 500, 70)] * 24, "8ELi1ELi4"),
    (10, [(500, 500, 70)] * 24, "8ELi1ELi4"), (11, [(500, 500, 70)] * 24, "4ELi2ELi2"),
    (6, [(100, 100, 70)], "2ELi2ELi1"), (6, [(100, 100, 70)] * 16, "4ELi1ELi4"),
    (5, [(300, 300, 270)] * 8, "4ELi1ELi4"),
    (6, [(150, 90, 70), (150, 90, 11200), (150, 90, 23000)], "4ELi1ELi4"),
    (7, [(33, 20, 9600), (33, 20, 20000), (33, 20, 129)], "4ELi2ELi2"),
    (6, [(900, 900, 11200), (40, 30, 129), (900, 900, 70), (900, 900, 11200)], "8ELi1ELi8"),
    (7, [(900, 900, 9600), (40, 30, 129), (900, 900, 70), (900, 900, 9600)], "8ELi1ELi4")])
def test_tiles_of_batches(child, s, sizes, tile):
    child(r"""
import numpy as np
s, sizes, tile = %d, %r, "%s"
n = len(sizes)
lib.ozaki_batched_graphs(0)
m, nn, k = (np.array(x, dtype=np.int64) for x in zip(*sizes))
one, zero = np.ones(n, dtype=np.complex128), np.zeros(n, dtype=np.complex128)
at, N = np.full(n, P, dtype=np.uint64), np.full(n, ord("N"), dtype=np.uint8)
sl, used = np.full(n, s, dtype=np.int32), np.zeros(n, dtype=np.int32)
p = lambda x: x.ctypes.data_as(ctypes.c_void_p)
assert lib.ozaki_zgemm_batched(p(N), p(N), p(m), p(nn), p(k), p(one), p(at), p(m), p(at), p(k), p(zero), p(at),
                               p(m), n, p(sl), p(used)) == 0
names = [l[1] for l in of(log(), "launch")]
assert any("k_ozgemmILi%%dELi%%s" %% (s, tile) in x for x in names), names
print("ok")
""" % (s, sizes, tile))
