"""GPU parity of the sample-level forward at the sizes where its bag kernel changes course: bags around one round of
64 lookups and around the four rounds of a workgroup, groups of lookups with one prefix around the largest that every
row of lanes gathers alike, averages on both sides of the rule that shares a bag among four wavefronts."""
import numpy as np
import pytest
import torch

import tt_workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank", [32, 64])
@pytest.mark.parametrize("lens", [(64, 64, 64, 64), (63, 65, 64, 63), (0, 257, 1, 255, 0), (1, 2, 5, 6, 7, 8, 9, 33), (1500,),
                                  (0, 0, 64)])
def test_bag_and_group_edges(ora, rank, lens):
    import gpu_util as g
    import paper_2507_14668_amd as tt
    print("case bag chains rank=%d lens=%s" % (rank, lens), flush=True)
    rng = np.random.default_rng(rank + sum(lens))
    n, nnz = (3, 4, 50), sum(lens)
    shape = wl.TableShape(n[0] * n[1] * n[2] - 1, n, (4, 8, 4), (1, rank, rank, 1))
    cores = [(0.2 * rng.standard_normal(shape.core_size(k))).astype(np.float32) for k in range(3)]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    for groups in (1, 9, 12):  # lookups per prefix: all of a bag, about seven, fewer
        idx = (rng.integers(0, groups, nnz) * n[2] + rng.integers(0, n[2] - 1, nnz)).astype(np.int64)
        idx[rng.random(nnz) < 0.05] = -1
        table = g.gpu_table(shape, cores)
        d_idx, d_off = torch.from_numpy(idx).cuda(), torch.from_numpy(off).cuda()
        plan = tt.tt_index_reorder(table, d_idx, d_off)
        out = tt.tt_emb_bag_forward_sample(table, plan, d_off)
        ref = ora.forward(shape, cores, np.where(idx < 0, shape.num_rows, idx), off)
        g.assert_close_rows(out.cpu().numpy(), ref, g.FWD_RTOL, shape.dim, "forward(sample)")
        assert torch.equal(tt.tt_emb_bag_forward_sample(table, plan, d_off), out)


@pytest.mark.parametrize("rank", [32, 64])
@pytest.mark.parametrize("lens", [(1,) * 37, (0,) * 9, (0, 1, 0, 0, 2, 0, 1), (0, 0, 63, 0, 1, 0), (0, 500, 0)])
def test_short_and_empty_bags(ora, rank, lens):
    """One-lookup bags, and empty ones, which leave before the sums over the lanes are formed: alone in the batch, between
    others in a workgroup, and as a bag of a workgroup's own."""
    test_bag_and_group_edges(ora, rank, lens)
