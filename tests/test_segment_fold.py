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
