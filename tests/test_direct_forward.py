"""The plan-free forward of short batches (emulated kernels) against the oracle and against reorder + planned forward: one and two
launches, empty bags, invalid lookups, offsets that are no CSR array, a table with fewer rows than the batch has lookups."""
import ctypes

import numpy as np
import pytest

import tt_workloads as wl
from test_cpu_emulation import BUILD_DIR, _aligned, _load, _ptr, _table, emu_build

pytestmark = pytest.mark.skipif(not emu_build.available(), reason="host clang++ of the ROCm toolchain not found")


@pytest.fixture(scope="module")
def emu():
    lib, binding = _load(emu_build.build_shared(BUILD_DIR))
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    lib.tt_emb_bag_forward_static.argtypes = [vp, vp, vp, i64, i64, vp, vp]
    return lib, binding


@pytest.mark.parametrize("r,n,lens,spoil", [
    (32, (5, 3, 7), (20,), ""), (64, (5, 3, 7), (0, 7, 0, 13), ""), (32, (5, 3, 7), (9, 0, 30, 8), ""),
    (64, (5, 3, 7), (3, 31), "indices"), (32, (5, 3, 7), (4, 20, 3), "indices"), (32, (5, 3, 7), (6, 10, 6, 4), "offsets"),
    (32, (5, 3, 7), (16, 10, 16, 14), "offsets"), (64, (2, 3, 2), (25, 15), "")])
def test_direct_forward_matches_oracle_and_plan(emu, ora, r, n, lens, spoil):
    import gpu_util as g
    lib, binding = emu
    shape, cores, _, _, _ = wl.small_random_problem(7, n=n, d=(4, 8, 4), r=(1, r, r, 1), sigma=0.2)
    rng = np.random.default_rng(len(lens) + r)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    nnz, nb = int(off[-1]), len(lens)
    idx = rng.integers(0, shape.num_rows, nnz).astype(np.int64)
    if spoil == "indices":
        idx[[1, 5, nnz - 1]] = (-1, shape.num_rows, 2 ** 40)
    if spoil == "offsets":
        off[1], off[3] = nnz + 5, -2
    cores = [np.ascontiguousarray(_aligned(c.nbytes).view(np.float32)) for c in cores]
    for c in cores:
        c[:] = 0.3 * rng.standard_normal(c.size)
    table = _table(binding, shape, cores)
    out = np.full((nb, shape.dim), np.nan, np.float32)
    assert lib.tt_emb_bag_forward_static(ctypes.byref(table), _ptr(idx), _ptr(off), nnz, nb, _ptr(out), None) == 0
    ws, plan = _aligned(lib.tt_workspace_bytes(ctypes.byref(table), nnz, nb)), binding.CPlan()
    assert lib.tt_index_reorder(ctypes.byref(table), _ptr(idx), _ptr(off), nnz, nb, None, _ptr(ws), ws.nbytes, ctypes.byref(plan), None) == 0
    ref = np.full_like(out, np.nan)
    assert lib.tt_emb_bag_forward(ctypes.byref(table), ctypes.byref(plan), _ptr(idx), _ptr(off), nnz, nb, _ptr(ref), None) == 0
    # (the host compiler may contract the emulated products and sums differently in the two kernels: bits are compared on the GPU)
    np.testing.assert_allclose(out, ref, rtol=0, atol=2e-6 * np.abs(ref).max())
    if not spoil:
        g.assert_close_rows(out, ora.forward(shape, cores, idx, off), g.FWD_RTOL, shape.dim, "direct forward")


# more bags than the one-launch route takes: two launches, no lookups at all, a plan (fewer rows than lookups)
@pytest.mark.parametrize("n,lens,spoil", [((5, 3, 7), (0,) * 90 + (7, 1, 12) + (0,) * 30, ""), ((5, 3, 7), (0,) * 120, "no lookups"),
                                          ((2, 3, 2), (0,) * 100 + (25, 5), "")])
def test_direct_forward_of_many_bags(emu, ora, n, lens, spoil):
    test_direct_forward_matches_oracle_and_plan(emu, ora, 64, n, lens, spoil)


@pytest.mark.parametrize("r,n,lens,spoil", [
    (32, (5, 3, 7), (20,), ""), (64, (5, 3, 7), (0, 7, 0, 13), ""), (32, (5, 3, 7), (300, 1, 40), ""), (64, (5, 3, 7), (3, 70), "indices"),
    (32, (5, 3, 7), (6, 10, 6, 4), "offsets"), (64, (2, 3, 2), (25, 15), ""), (32, (5, 3, 7), (), "")])
def test_direct_bf16_forward_matches_oracle_and_plan(emu, ora, r, n, lens, spoil):
    import gpu_util as g
    from test_gpu_parity_small import round_to_bf16
    lib, binding = emu
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    lib.tt_cores_to_bf16.argtypes = [vp, vp, ctypes.c_size_t, vp]
    lib.tt_bf16_cores_bytes.restype, lib.tt_bf16_cores_bytes.argtypes = ctypes.c_size_t, [vp]
    lib.tt_emb_bag_forward_bf16.argtypes = [vp, vp, vp, vp, i64, i64, vp, vp]
    lib.tt_emb_bag_forward_bf16_direct.argtypes = [vp, vp, vp, vp, i64, i64, vp, vp]
    lib.tt_forward_bf16_direct_pays.argtypes = [vp, i64, i64]
    shape, cores, _, _, _ = wl.small_random_problem(9, n=n, d=(4, 8, 4), r=(1, r, r, 1), sigma=0.2)
    rng = np.random.default_rng(len(lens) + r)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    nnz, nb = int(off[-1]), len(lens)
    idx = rng.integers(0, shape.num_rows, nnz).astype(np.int64)
    if spoil == "indices":
        idx[[1, 5, nnz - 1]] = (-1, shape.num_rows, 2 ** 40)
    if spoil == "offsets":
        off[1], off[3] = nnz + 5, -2
    raw = cores
    cores = [_aligned(np.asarray(c).size * 4).view(np.float32) for c in raw]
    for c, x in zip(cores, raw):
        c[:] = np.asarray(x, np.float32).reshape(-1)
    table = _table(binding, shape, cores)
    bf = _aligned(lib.tt_bf16_cores_bytes(ctypes.byref(table)))
    assert lib.tt_cores_to_bf16(ctypes.byref(table), _ptr(bf), bf.nbytes, None) == 0
    out = np.full((nb, shape.dim), np.nan, np.float32)
    assert lib.tt_emb_bag_forward_bf16_direct(ctypes.byref(table), _ptr(bf), _ptr(idx), _ptr(off), nnz, nb, _ptr(out), None) == 0
    assert lib.tt_forward_bf16_direct_pays(ctypes.byref(table), nnz, nb) == 1
    assert lib.tt_forward_bf16_direct_pays(ctypes.byref(table), nnz, -1) == 0
    assert lib.tt_forward_bf16_direct_pays(ctypes.byref(table), 10 ** 6, 1000) == 0
    ws, plan = _aligned(lib.tt_workspace_bytes(ctypes.byref(table), nnz, nb)), binding.CPlan()
    assert lib.tt_index_reorder(ctypes.byref(table), _ptr(idx), _ptr(off), nnz, nb, None, _ptr(ws), ws.nbytes, ctypes.byref(plan), None) == 0
    ref = np.full_like(out, np.nan)
    assert lib.tt_emb_bag_forward_bf16(ctypes.byref(table), _ptr(bf), ctypes.byref(plan), _ptr(off), nnz, nb, _ptr(ref), None) == 0
    if nb == 0:
        return
    # both are fp32 sums of the same products, over chains of at most 300 lookups in another order
    np.testing.assert_allclose(out, ref, rtol=0, atol=5e-6 * np.abs(ref).max())
    if not spoil:
        g.assert_close_rows(out, ora.forward(shape, [round_to_bf16(c) for c in raw], idx, off), g.FWD_RTOL, shape.dim, "direct bf16 forward")


def test_direct_bf16_forward_of_the_last_lookups_of_2_31(tmp_path):
    """A bag that ends where 32-bit positions end (compiled so that they wrap).  In a process of its own: the indices are a sparse file of 16 GB of which the bag's
    pages are touched, and reading elsewhere ends the process."""
    import subprocess
    import sys
    script = """
import ctypes, sys
import numpy as np
sys.path[:0] = %r
import tt_workloads as wl
from test_cpu_emulation import BUILD_DIR, _aligned, _load, _ptr, _table, emu_build
lib, binding = _load(%r)
vp, i64 = ctypes.c_void_p, ctypes.c_int64
lib.tt_cores_to_bf16.argtypes = [vp, vp, ctypes.c_size_t, vp]
lib.tt_bf16_cores_bytes.restype, lib.tt_bf16_cores_bytes.argtypes = ctypes.c_size_t, [vp]
lib.tt_emb_bag_forward_bf16_direct.argtypes = [vp, vp, vp, vp, i64, i64, vp, vp]
shape, raw, _, _, _ = wl.small_random_problem(9, n=(5, 3, 7), d=(4, 8, 4), r=(1, 32, 32, 1), sigma=0.2)
cores = [_aligned(np.asarray(c).size * 4).view(np.float32) for c in raw]
for c, x in zip(cores, raw):
    c[:] = np.asarray(x, np.float32).reshape(-1)
table = _table(binding, shape, cores)
bf = _aligned(lib.tt_bf16_cores_bytes(ctypes.byref(table)))
assert lib.tt_cores_to_bf16(ctypes.byref(table), _ptr(bf), bf.nbytes, None) == 0
rng, out = np.random.default_rng(0), []
last = rng.integers(0, shape.num_rows, 300)
for nnz in (300, 2 ** 31 - 2):
    idx = np.memmap(%r, np.int64, "w+", shape=(nnz,))
    idx[-300:] = last
    off = np.array([nnz - 300, nnz], np.int64)
    out.append(np.full(shape.dim, np.nan, np.float32))
    assert lib.tt_emb_bag_forward_bf16_direct(ctypes.byref(table), _ptr(bf), _ptr(idx), _ptr(off), nnz, 1, _ptr(out[-1]), None) == 0
assert np.array_equal(*out) and np.isfinite(out[0]).all()
""" % ([p for p in sys.path if p], emu_build.build_shared(BUILD_DIR, "wrap", ["-fwrapv"]), str(tmp_path / "indices"))
    res = subprocess.run([sys.executable, "-c", script], capture_output=True, text=True, timeout=300)
    (tmp_path / "indices").unlink(missing_ok=True)
    assert res.returncode == 0, res.stderr[-2000:]


# which way the module goes, on both sides of every limit: short sums of costs, and at ranks 64 one or two bags with all lookups
@pytest.mark.parametrize("r,nnz,bags,pays", [
    (32, 0, 0, 1), (32, 2048, 300, 1), (32, 46000, 1, 1), (32, 46000, 900, 1), (32, 47400, 900, 0), (32, 50, 9000, 1), (32, 50, 9300, 0),
    (64, 1000, 1, 1), (64, 1001, 1, 0), (64, 5000, 1, 0), (64, 6000, 2, 1), (64, 6001, 2, 0), (64, 14000, 3, 1), (64, 14600, 3, 0),
    (64, 2048, 300, 1), (64, 20000, 2000, 0)])
def test_where_the_bf16_forward_goes_without_a_plan(emu, r, nnz, bags, pays):
    lib, binding = emu
    lib.tt_forward_bf16_direct_pays.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64]
    shape = wl.TableShape(105, (5, 3, 7), (4, 8, 4), (1, r, r, 1))
    table = _table(binding, shape, [np.zeros(4, np.float32)] * 3)
    assert lib.tt_forward_bf16_direct_pays(ctypes.byref(table), nnz, bags) == pays
