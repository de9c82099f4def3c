"""Tables with so many slices that one workgroup per slice and tile is more than a launch holds (2^32 threads): the call
is served all the same, and every slice of the gradient is written."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_core1_gradient_of_many_slices():
    """8.4 million i2 with two column tiles each: a workgroup for each of them would be 16.8 million."""
    import gpu_util as g
    import paper_2507_14668_amd as tt
    n, d, r = (1, 8_400_000, 1), (2, 5, 2), (1, 1, 13, 1)
    print("case wide grid n=%s d=%s r=%s" % (n, d, r), flush=True)
    rng = np.random.default_rng(8)
    idx = np.concatenate([[0, 1, n[1] - 1, n[1] // 2, n[1] // 2 - 1], rng.integers(0, n[1], 200), [7] * 9]).astype(np.int64)
    u = np.unique(idx)
    off = np.arange(len(idx) + 1, dtype=np.int64)
    grad = rng.standard_normal((len(idx), d[0], d[1], d[2])).astype(np.float32)
    g1, g3 = (0.5 * rng.standard_normal(s).astype(np.float32) for s in ((d[0],), (r[2], d[2])))
    g2 = (0.5 * rng.standard_normal((len(u), d[1], r[2]))).astype(np.float32)
    core1 = torch.zeros(n[1], d[1] * r[2], device="cuda")
    core1[torch.from_numpy(u).cuda()] = torch.from_numpy(g2).view(len(u), -1).cuda()
    table = tt.Table(n[1], n, d, r, [torch.from_numpy(g1).cuda(), core1.view(-1), torch.from_numpy(g3).view(-1).cuda()])
    d_idx, d_off, d_grad = (torch.from_numpy(x).cuda() for x in (idx, off, grad.reshape(len(idx), -1)))
    plan = tt.tt_index_reorder(table, d_idx, d_off)
    dcores = [torch.full_like(c, float("nan")) for c in table.cores]
    tt.tt_emb_bag_backward(table, plan, d_idx, d_off, d_grad, dcores=dcores)
    merged = np.zeros((len(u),) + d)
    np.add.at(merged, np.searchsorted(u, idx), grad.astype(np.float64))
    ref = np.einsum("a,uabc,sc->ubs", g1.astype(np.float64), merged, g3.astype(np.float64))
    got = dcores[1].view(n[1], -1)
    g.assert_close_rows(got[torch.from_numpy(u).cuda()].cpu().numpy(), ref.reshape(len(u), -1), g.GRAD_RTOL, d[1] * r[2], "dG2")
    assert int(torch.count_nonzero(got.any(dim=1))) == len(u) and not bool(torch.isnan(got).any())  # zeros everywhere else
    del dcores, got
    tt.tt_emb_bag_backward_sgd(table, plan, d_idx, d_off, d_grad, 0.25)
    new = g2.astype(np.float64) - 0.25 * ref
    g.assert_close_rows(core1[torch.from_numpy(u).cuda()].cpu().numpy(), new.reshape(len(u), -1), g.GRAD_RTOL, d[1] * r[2], "G2")
    assert int(torch.count_nonzero(core1.any(dim=1))) == len(u)
