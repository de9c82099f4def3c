"""GPU parity of the matrix-core kernels where a chunk of eight prefixes is partly filled: four or fewer take one row
tile at rank 64, as the only chunk of an i2, as the last of several, and as one part of a split i2."""
import numpy as np
import pytest

import tt_workloads as wl
from test_gpu_parity_small import g, run_all  # noqa: F401  (g is the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [32, 64])
@pytest.mark.parametrize("n1", [1, 3, 4, 5, 8, 9, 12, 13, 68])
def test_prefixes_per_chunk(g, ora, rank, n1):  # noqa: F811
    print("case chunk fill rank=%d n1=%d" % (rank, n1), flush=True)
    shape, cores, idx, off, grad = wl.small_random_problem(500 + n1, n=(n1, 2, 3), d=(4, 8, 4), r=(1, rank, rank, 1),
                                                          num_bags=6 * n1 + 3, max_len=3, sigma=0.2)
    idx[:6 * n1] = np.resize(np.arange(6 * n1), len(idx[:6 * n1]))  # every prefix, as far as the lookups reach
    run_all(g, ora, shape, cores, idx, off, grad)
