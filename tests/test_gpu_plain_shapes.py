"""GPU parity of the backward kernel that gives one wavefront a distinct prefix (shapes without a matrix-core kernel and
with small operands) and of the core-1 reduction behind them, at the sizes where their loops change: rows per
prefix around the solo limit and the batch of four, ranks around sixteen, column tiles of 64, five values of j1,
chunks of 64 (prefix, j1) pairs, and the first shape that is too large for them."""
import pytest

import tt_workloads as wl
from test_gpu_parity_small import g, run_all  # noqa: F401  (g is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,n,d,r,nb", [
    (11, (3, 5, 16), (2, 2, 4), (1, 4, 4, 1), 900),      # 16 rows per prefix: one wavefront each
    (12, (3, 5, 17), (2, 2, 4), (1, 4, 4, 1), 900),      # 17: all four wavefronts, the last batch has one row
    (13, (2, 3, 130), (4, 4, 4), (1, 16, 16, 1), 2500),  # 130 rows per prefix
    (14, (40, 4, 3), (5, 3, 2), (1, 17, 5, 1), 1500),    # five values of j1, 17 of r1; 200 (prefix, j1) pairs per i2
    (15, (13, 7, 5), (2, 4, 6), (1, 12, 20, 1), 600),    # 80 columns: two column tiles; d3 that no float4 divides
    (16, (32, 2, 2), (2, 3, 3), (1, 31, 7, 1), 700),     # exactly 64 pairs per i2; two r1 tiles, the second partly filled
    (17, (33, 2, 2), (2, 3, 3), (1, 33, 7, 1), 700),     # 66 pairs; three r1 tiles
    (18, (5, 3, 20), (1, 1, 1), (1, 1, 1, 1), 300),      # one column of everything
    (19, (6, 3, 20), (4, 4, 4), (1, 32, 32, 1), 400),    # too large for a wavefront: workgroup per prefix
])
def test_wavefront_per_prefix_shapes(g, ora, seed, n, d, r, nb):  # noqa: F811
    print("case plain shapes seed=%d n=%s d=%s r=%s" % (seed, n, d, r), flush=True)
    run_all(g, ora, *wl.small_random_problem(seed, n=n, d=d, r=r, num_bags=nb, max_len=4))
