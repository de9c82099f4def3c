"""The matrix-core forward on split fp32 numbers, above the sizes of the direct forward: error against 64 bits with cores of very
different sizes, infinities, NaN and the largest numbers against the arm without a plan, by both routes that use it."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _case(tt, r, n, spread, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    d, rr, rows = (4, 8, 4), (1, r, r, 1), n[0] * n[1] * n[2]
    cores = []
    for k in range(3):
        m = rr[k] * n[k] * d[k] * rr[k + 1]
        c = 0.2 * torch.randn(m, device="cuda", generator=g)
        cores.append(c * 10.0 ** (spread * (2 * torch.rand(m, device="cuda", generator=g) - 1)))
    nnz = 16385 if r == 32 else 8193  # the first size above the direct forward's
    idx = torch.randint(0, rows, (nnz,), device="cuda", generator=g)
    off = torch.cat([torch.arange(0, nnz, 3, device="cuda"), torch.tensor([nnz], device="cuda")])
    return tt.Table(rows, n, d, rr, cores), idx, off


def _exact(table, cores, idx, off):
    n, d, r = table.n, table.d, table.r
    c = [x.double().view(r[k], n[k], d[k], r[k + 1]) for k, x in enumerate(cores)]
    u, inv = torch.unique(idx, return_inverse=True)
    pu, pinv = torch.unique(u // n[2], return_inverse=True)
    a = c[0][0, pu // n[1]]
    b = c[1][:, pu % n[1]].permute(1, 0, 2, 3).reshape(len(pu), r[1], -1).contiguous()
    p12 = torch.bmm(a, b).view(len(pu), d[0] * d[1], r[2])
    rows = torch.bmm(p12[pinv], c[2][:, u % n[2], :, 0].permute(1, 0, 2).contiguous()).view(len(u), -1)
    bag = torch.repeat_interleave(torch.arange(off.numel() - 1, device="cuda"), off[1:] - off[:-1])
    return torch.zeros(off.numel() - 1, table.dim, dtype=torch.float64, device="cuda").index_add_(0, bag, rows[inv])


def _routes(tt, table, idx, off):
    plan = tt.tt_index_reorder(table, idx, off)
    return tt.tt_emb_bag_forward(table, plan, idx, off), tt.tt_emb_bag_forward_sample(table, plan, off)


# prefixes per i2: up to 3 (half tiles), 8 (one chunk), 13, and 70 (the staged plan entries are refilled)
@pytest.mark.parametrize("r", [32, 64])
@pytest.mark.parametrize("n", [(3, 300, 40), (8, 61, 20), (13, 11, 30), (70, 9, 8)])
@pytest.mark.parametrize("spread", [0, 3])
def test_error_against_64_bits(r, n, spread):
    import paper_2507_14668_amd as tt
    print("case split r=%d n=%s spread=%d" % (r, n, spread), flush=True)
    table, idx, off = _case(tt, r, n, spread, r + n[0])
    want, size = _exact(table, table.cores, idx, off), _exact(table, [c.abs() for c in table.cores], idx, off)
    for out in _routes(tt, table, idx, off):
        # two sums of r terms and one of three rows, two roundings a path and 2^-24 for the terms left out, twice over
        assert bool(((out.double() - want).abs() <= 2 * (2 * r + 6) * 2.0 ** -24 * size).all())


@pytest.mark.parametrize("r", [32, 64])
@pytest.mark.parametrize("core", [0, 1, 2])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.4e38])
def test_infinities_nan_and_the_largest_numbers(r, core, value):
    import paper_2507_14668_amd as tt
    print("case split r=%d core=%d value=%s" % (r, core, value), flush=True)
    table, idx, off = _case(tt, r, (13, 11, 30), 0, 7)
    for c in table.cores:
        c.mul_(0.25)  # sums of products with 3.4e38 stay finite in every order
    table.cores[core][[3, table.cores[core].numel() // 2]] = value
    want = tt.tt_emb_bag_forward(table, None, idx, off)
    assert bool(torch.isfinite(want).all()) == (value == 3.4e38)
    fin = torch.isfinite(want)
    for route, out in enumerate(_routes(tt, table, idx, off)[:1 if core == 2 else 2]):
        assert torch.equal(torch.isfinite(out), fin)
        # (the sample route adds core-2 slices first: an infinity times a sum is not the sum of two infinities, and two of the
        # largest numbers overflow)
        assert route == 1 or torch.equal(torch.isnan(out), torch.isnan(want))
        assert torch.allclose(out[fin], want[fin], rtol=1e-4, atol=1e-5 * float(want[fin].abs().max()))
