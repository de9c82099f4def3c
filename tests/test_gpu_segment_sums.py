"""The two-stage core-0 sum at the widest slice that a table may have (d1 * R1 = 4096): its lane groups' sums take 64 KB of LDS
by themselves, with few chunks and with as many as make shorter vectors take a chunk per lane group."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n2", [5000, 60000])
def test_widest_core0_slices(n2):
    import paper_2507_14668_amd as tt
    print("case widest core-0 slice n2=%d" % n2, flush=True)
    d, r, n = (32, 1, 1), (1, 128, 1, 1), (1, n2, 1)
    g = torch.Generator(device="cuda").manual_seed(n2)
    cores = [torch.randn(r[k] * n[k] * d[k] * r[k + 1], device="cuda", generator=g) for k in range(3)]
    table = tt.Table(n2, n, d, r, cores)
    idx = torch.randperm(n2, device="cuda", generator=g)
    off = torch.arange(n2 + 1, device="cuda")
    grad = torch.randn((n2, 32), device="cuda", generator=g)
    plan = tt.tt_index_reorder(table, idx, off)
    out = tt.tt_emb_bag_forward(table, plan, idx, off)
    dg = tt.tt_emb_bag_backward(table, plan, idx, off, grad)
    a, b, c = (x.double() for x in table.cores)
    a, b = a.view(32, 128), b.view(128, n2)[:, idx]  # (one slice of core 0, one number of core 2)
    g64 = grad.double()
    want = [c * (b @ g64).t().reshape(-1), torch.zeros(128, n2, dtype=torch.float64, device="cuda"), ((b.t() @ a.t()) * g64).sum()]
    want[1][:, idx] = c * (g64 @ a).t()
    assert torch.allclose(out.double(), c * (b.t() @ a.t()), rtol=0, atol=1e-4)
    for x, y in zip(dg, want):  # sums of up to 60000 terms of one size, in two levels and more: far below 1e-5 of the largest
        assert float((x.double() - y.reshape(-1)).abs().max()) <= 1e-5 * float(y.abs().max()) + 1e-3 * (x.numel() == 1)
