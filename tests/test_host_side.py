"""The library's host code without a GPU: in a process of its own, on a stand-in for the HIP runtime whose kernels do nothing
(host_runtime.cpp)."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_1102_3828_amd", "libivfadcr.so")

HEAD = """
import ctypes as C, numpy as np, sys
rt = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # in front of the library's own runtime
rt.host_live_bytes.restype = C.c_size_t
lib = C.CDLL(sys.argv[2])
lib.ivfr_last_error.restype = C.c_char_p
i64, u64, vp = C.c_int64, C.c_uint64, C.c_void_p
OOM = -3
class Params(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("d", "c", "m", "m_refine", "device")]
def create(d, c, m, mr):
    p, h = Params(d, c, m, mr, 0), vp()
    assert lib.ivfr_create(C.byref(p), C.byref(h)) == 0, lib.ivfr_last_error()
    return p, h
def ptr(a): return None if a is None else a.ctypes.data_as(vp)
def books(p):
    f = lambda *s: np.zeros(s, np.float32)
    return f(p.c, p.d), f(p.m, 256, p.d // p.m), f(p.m_refine, 256, p.d // p.m_refine) if p.m_refine else None
def set_books(p, h): return lib.ivfr_set_codebooks(h, *map(ptr, books(p)))
def train(p, h, n, iters=1):
    x = np.zeros((n, p.d), np.uint8)
    return lib.ivfr_train(h, ptr(x), i64(n), C.c_int32(iters), u64(1))
def add(p, h, n, base):
    x = np.zeros((n, p.d), np.uint8)
    return lib.ivfr_add(h, ptr(x), i64(n), i64(base))
def required(p, N):
    ib = i64()
    assert lib.ivfr_memory_required(C.byref(p), i64(N), i64(0), 1, 1, i64(0), C.byref(ib), None) == 0
    return ib.value
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rt") / "libhost_runtime.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "host_runtime.cpp"), "-o", so], check=True)
    return so


def _run(runtime, code):
    r = subprocess.run([sys.executable, "-c", HEAD + code, runtime, LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("d,c,m,mr", [(128, 300, 8, 16), (64, 2000, 16, 0), (512, 9, 16, 16)])
def test_codebooks_after_a_failed_allocation(runtime, d, c, m, mr):
    """Whichever array could not be allocated: nothing is kept, and the same call made again has all of them."""
    _run(runtime, f"""
shape = ({d}, {c}, {m}, {mr})
p, h = create(*shape)
empty = rt.host_live_bytes()
assert set_books(p, h) == 0
whole = rt.host_live_bytes() - empty
lib.ivfr_destroy(h)
failed = 0
for n in range(64):
    for call in (set_books, lambda p, h: train(p, h, max(p.c, 256))):
        p, h = create(*shape)
        empty = rt.host_live_bytes()
        rt.host_fail_allocation(n)
        rc = call(p, h)
        rt.host_fail_allocation(-1)
        held = rt.host_live_bytes() - empty
        assert rc in (0, OOM) and held in (0, whole), (n, rc, held, whole)
        assert held == whole or rc == OOM
        failed += rc == OOM
        assert set_books(p, h) == 0 and rt.host_live_bytes() - empty == whole, n
        lib.ivfr_destroy(h)
assert failed > 12 and rt.host_live_bytes() == 0
""")


@pytest.mark.parametrize("d,c,m,mr,n", [(128, 256, 8, 8, 5000), (512, 1024, 16, 16, 300), (64, 1025, 16, 0, 70), (32, 1, 32, 8, 1), (256, 300, 64, 64, 999),
                                        (8, 20000, 4, 4, 0)])
def test_memory_required_covers_what_an_index_holds(runtime, d, c, m, mr, n):
    """At most the stated bytes, which are above what is held by no more than the largest possible padding of lists (and the fill
    counts that only a built index has)."""
    _run(runtime, f"""
p, h = create({d}, {c}, {m}, {mr})
n = {n}
assert set_books(p, h) == 0
offsets = np.full(p.c + 1, n, np.int64)        # all in the first list
offsets[0] = 0
ids, codes, rcodes = np.arange(n, dtype=np.int32), np.zeros((n, p.m), np.uint8), np.zeros((n, max(p.m_refine, 1)), np.uint8)
assert lib.ivfr_import(h, i64(n), ptr(offsets), ptr(ids), ptr(codes), ptr(rcodes)) == 0, lib.ivfr_last_error()
held, need = rt.host_live_bytes(), required(p, n)
record = max(32, 1 << (p.m + p.m_refine + 7).bit_length()) if p.m + p.m_refine + 8 <= 128 else 192
assert held <= need <= held + 31 * p.c * (p.m + record) + 8 * p.c + 256, (held, need)
lib.ivfr_destroy(h)
assert rt.host_live_bytes() == 0
""")


def test_function_attributes_are_set_when_an_index_is_created(runtime):
    """A function's largest dynamic LDS belongs to the process: calls of two indexes in two threads would take it from one another."""
    _run(runtime, """
a, b = create(8, 16384, 4, 4), create(128, 13000, 4, 0)      # (largest counters; sub-vectors of 2 dimensions and of 32)
before = rt.host_attributes()
for i in range(2):
    for p, h in (a, b):
        assert train(p, h, 16384) == 0
for i in range(2):
    for p, h in (a, b):
        assert add(p, h, 3000, 3000 * i) == 0
assert rt.host_attributes() == before > 0
""")


@pytest.mark.parametrize("m", [4, 8, 16, 32, 64])
def test_every_small_call_has_its_kernel(runtime, m):
    """Calls that run one workgroup per query, in every shape that they are launched in: dimensions, tables (loaded, split, computed),
    a query to a compute unit and more, one group of lists and several."""
    _run(runtime, f"""
m = {m}
x, ids, dist = np.zeros((700, 2048), np.float32), np.zeros(700 * 100, np.int32), np.zeros(700 * 100, np.float32)
for d in [8 << i for i in range(9) if 8 << i <= 32 * m and (8 << i) >= m]:
    p, h = create(d, 70, m, 0)
    assert set_books(p, h) == 0
    n = 70 * 50
    assert lib.ivfr_import(h, i64(n), ptr(np.arange(71, dtype=np.int64) * 50), ptr(np.arange(n, dtype=np.int32)), ptr(np.zeros((n, m), np.uint8)), None) == 0
    for mode in (0, 1):
        assert lib.ivfr_set_table_mode(h, mode) == 0
        for nq in (1, 256, 257, 700):
            for w in (1, 3, 5, 8, 64):
                for kp in (1, 100):
                    rc = lib.ivfr_search(h, ptr(x), i64(nq), w, kp, 1, ptr(ids), ptr(dist), None)
                    assert rc == 0, (d, mode, nq, w, kp, lib.ivfr_last_error())
    lib.ivfr_destroy(h)
""")
