"""GPU parity of the index-reorder plan where its launches change shape: batches around one wavefront and
one workgroup (plan built by a single workgroup), around one sort tile, one group of tiles and the limits
of both ways of adding up tile counts.  Integer work: bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import tt_workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nnz", [1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 3072, 32 * 1024 + 1,
                                 64 * 1024, 64 * 1024 + 1, 96 * 1024 - 1, 1024 * 1024, 1024 * 1024 + 1])
def test_plan_at_tile_edges(ora, nnz):
    import gpu_util as g
    import paper_2507_14668_amd as tt
    print("case plan nnz=%d" % nnz, flush=True)
    rng = np.random.default_rng(nnz)
    n = [(7, 9, 11), (61, 67, 63), (1, 1, 500), (300, 1023, 1)][nnz % 4]
    shape = wl.TableShape(n[0] * n[1] * n[2] - nnz % 2, n, (2, 2, 2), (1, 2, 2, 1))
    cores = [np.zeros(shape.core_size(k), np.float32) for k in range(3)]
    # runs of equal rows (skewed), empty bags, lookups outside the table
    idx = np.minimum((shape.num_rows ** rng.random(nnz)).astype(np.int64) - 1, shape.num_rows - 1)
    idx[rng.random(nnz) < 0.01] = -1
    idx[rng.random(nnz) < 0.01] = shape.num_rows
    for bags in (1, max(1, nnz // 3), min(3 * nnz, 40_000)):
        cuts = np.sort(rng.integers(0, nnz + 1, bags - 1))
        off = np.concatenate([[0], cuts, [nnz]]).astype(np.int64)
        plan = tt.tt_index_reorder(g.gpu_table(shape, cores), torch.from_numpy(idx).cuda(), torch.from_numpy(off).cuda())
        g.assert_plan_equals_oracle(ora, shape, plan, idx, off)
    none = np.full(nnz, -1, np.int64)  # not one valid lookup
    plan = tt.tt_index_reorder(g.gpu_table(shape, cores), torch.from_numpy(none).cuda(), torch.from_numpy(off).cuda())
    g.assert_plan_equals_oracle(ora, shape, plan, none, off)
