"""Stage 2 of the two-stage segmented sums: the route with a chunk per lane group leaves the bits of the route with a chunk
per workgroup (the library's kernels compiled for the CPU, the second route for every size in a variant of its own)."""
import ctypes

import numpy as np
import pytest

import test_cpu_emulation as te
import tt_workloads as wl

pytestmark = te.pytestmark


@pytest.fixture(scope="module")
def routes():
    two_stage = "-DTT_SEG_WHOLE_MAX_AVG=-1"  # the core sums too, with their zero-filled slices
    return [te._load(te.emu_build.build_shared(te.BUILD_DIR, "fold", [two_stage])),
            te._load(te.emu_build.build_shared(te.BUILD_DIR, "spread", [two_stage, "-DTT_SEG2_SPREAD_CHUNKS=-1"]))]


@pytest.mark.parametrize("n,d,r,nb,ml", [
    ((2, 1, 2), (4, 8, 4), (1, 32, 32, 1), 700, 4),    # D = 128, eight lane groups: segments of hundreds of chunks
    ((2, 2, 40), (4, 8, 4), (1, 32, 32, 1), 500, 4),   # ... and of a few
    ((1, 2, 2), (2, 3, 2), (1, 3, 5, 1), 900, 3),      # D = 12, 64 lane groups
    ((1, 1, 3), (3, 3, 5), (1, 3, 5, 1), 600, 3),      # odd widths, one float a lane, four lane groups
    ((7, 5, 4), (1, 1, 1), (1, 2, 3, 1), 300, 5),      # D = 1, a lane group per thread
    # slices without lookups beside one that has them all, by i3 and by i1 (zero-filled, dense gradients)
    ((1, 2, 5000), (2, 3, 2), (1, 3, 5, 1), 40, 3),
])
def test_chunk_per_lane_group_equals_chunk_per_workgroup(routes, n, d, r, nb, ml):
    shape, cores, idx, off, grad = wl.small_random_problem(77, n=n, d=d, r=r, num_bags=nb, max_len=ml, sigma=0.2)
    a, b = (te._run(lib, shape, cores, idx, off, grad, 0.05) for lib in routes)
    for x, y in zip(a["plan"][1] + a["fused"] + a["updated"], b["plan"][1] + b["fused"] + b["updated"]):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("r", [32, 64])
def test_core_sums_into_unaligned_gradients(r):
    """Two and four strips a prefix with four-byte stores (gradient buffers off the 16-byte grid): whole segments by rounds and
    one position after the other, as the aligned sums up to the order of additions."""
    lib, binding = te._load(te.emu_build.build_shared(te.BUILD_DIR))
    shape, cores, idx, off, grad = wl.small_random_problem(31, n=(3, 5, 7), d=(4, 8, 4), r=(1, r, r, 1), num_bags=60, max_len=3, sigma=0.2)
    cores = [np.ascontiguousarray(c, dtype=np.float32) for c in cores]
    aligned = [te._aligned(4 * c.size).view(np.float32) for c in cores]
    for a, c in zip(aligned, cores):
        a[:] = c
    idx, off = np.ascontiguousarray(idx, dtype=np.int64), np.ascontiguousarray(off, dtype=np.int64)
    grad = np.ascontiguousarray(grad, dtype=np.float32)
    nnz, nb = len(idx), len(off) - 1
    table = te._table(binding, shape, aligned)
    ws = te._aligned(lib.tt_workspace_bytes(ctypes.byref(table), nnz, nb))
    plan = binding.CPlan()
    assert lib.tt_index_reorder(ctypes.byref(table), te._ptr(idx), te._ptr(off), nnz, nb, None, te._ptr(ws), ws.nbytes,
                                ctypes.byref(plan), None) == 0
    got = []
    for shift in (0, 1):
        dg = [te._aligned(4 * c.size + 16).view(np.float32)[shift:shift + c.size] for c in cores]
        arr = (ctypes.c_void_p * 3)(*[x.ctypes.data for x in dg])
        assert lib.tt_emb_bag_backward(ctypes.byref(table), ctypes.byref(plan), te._ptr(idx), te._ptr(off), nnz, nb, te._ptr(grad),
                                       arr, None) == 0
        got.append([x.copy() for x in dg])
    for x, y in zip(*got):
        assert np.allclose(x, y, rtol=0, atol=1e-6 * np.abs(x).max())


@pytest.fixture(scope="module")
def emu():
    return te._load(te.emu_build.build_shared(te.BUILD_DIR))


@pytest.mark.parametrize("n,d,r,nnz,rounds", [
    ((8, 8, 2), (2, 4, 6), (1, 12, 20, 1), 63, False), ((8, 8, 2), (2, 4, 6), (1, 12, 20, 1), 64, True),  # one strip: rows per i3
    ((1, 40, 4), (2, 3, 2), (1, 4, 8, 1), 31, False), ((1, 40, 4), (2, 3, 2), (1, 4, 8, 1), 32, True),    # prefixes per i1
    ((9, 9, 3), (4, 8, 4), (1, 32, 32, 1), 134, False), ((9, 9, 3), (4, 8, 4), (1, 32, 32, 1), 135, True),  # two strips
    ((9, 9, 3), (4, 8, 4), (1, 64, 64, 1), 135, False),                                                     # four
])
def test_whole_segments_by_rounds_from_a_length_on(emu, capfd, monkeypatch, n, d, r, nnz, rounds):
    """Which batches' whole segments go in rounds, and the gradients of both ways against 64 bits."""
    launches, dg, ref = te._backward_with_trace(emu, capfd, monkeypatch, n, d, r, nnz)
    assert [("true" in ln.split("k_seg_whole", 1)[1]) for ln in launches if "k_seg_whole" in ln] == [rounds], launches
    for a, b in zip(dg, ref):  # sums of up to 135 terms in 32 bits
        assert np.linalg.norm(a - b) <= 2e-6 * np.linalg.norm(b)
