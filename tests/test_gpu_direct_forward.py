"""Short batches of the allocation-free forward are summed without a plan (one launch up to 32 lookups, two up to 16384 or
8192): bit for bit the result of tt_index_reorder + tt_emb_bag_forward, on both sides of every limit, with invalid lookups, empty
and malformed bags, repeated rows, and replayed from a graph.  The bf16 inference forward without a plan against the planned one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _table(tt, r, rows=None, n=(60, 50, 40)):
    g = torch.Generator(device="cuda").manual_seed(r)
    d, rr = (4, 8, 4), (1, r, r, 1)
    cores = [0.2 * torch.randn(rr[k] * n[k] * d[k] * rr[k + 1], device="cuda", generator=g) for k in range(3)]
    return tt.Table(rows or n[0] * n[1] * n[2] - 7, n, d, rr, cores)


def _batch(rows, nnz, bags, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    idx = (rows ** torch.rand(nnz, device="cuda", dtype=torch.float64, generator=g)).long().clamp(max=rows - 1)
    if nnz > 8:  # invalid lookups among the others
        idx[nnz // 3], idx[nnz // 2], idx[-1] = -1, rows, 2 ** 40
    cut = torch.sort(torch.randint(0, nnz + 1, (bags - 1,), device="cuda", generator=g)).values
    ends = torch.tensor([nnz], device="cuda")
    return idx, torch.cat([torch.zeros_like(ends), cut, ends])


@pytest.mark.parametrize("r,nnz,bags", [
    (r, nnz, bags) for r, top in ((32, 16384), (64, 8192))
    for nnz, bags in ((0, 3), (1, 1), (9, 9), (31, 2), (32, 1), (32, 90), (33, 1), (33, 5), (64, 1), (257, 100), (2049, 300),
                      (top, 2000), (top + 1, 2000))])
def test_same_bits_as_with_a_plan(r, nnz, bags):
    import paper_2507_14668_amd as tt
    print("case direct r=%d nnz=%d bags=%d" % (r, nnz, bags), flush=True)
    table = _table(tt, r)
    idx, off = _batch(table.num_rows, nnz, bags, nnz + bags)
    out = torch.full((bags, 128), float("nan"), device="cuda")
    tt.tt_emb_bag_forward_static(table, idx, off, out)
    plan = tt.tt_index_reorder(table, idx, off)
    assert torch.equal(out, tt.tt_emb_bag_forward(table, plan, idx, off))


# few lookups in many bags: on both sides of the limits of the one-launch route (768 bags at ranks 32, 96 at ranks 64), up to the
# most bags that are served without a plan and one more; a table with fewer rows than the batch has lookups
@pytest.mark.parametrize("r", [32, 64])
@pytest.mark.parametrize("nnz", [0, 1, 20, 32])
@pytest.mark.parametrize("bags", [96, 97, 768, 769, 16384, 16385])
@pytest.mark.parametrize("small", [False, True])
def test_few_lookups_in_many_bags(r, nnz, bags, small):
    import paper_2507_14668_amd as tt
    print("case direct r=%d nnz=%d bags=%d small=%d" % (r, nnz, bags, small), flush=True)
    table = _table(tt, r, rows=17, n=(2, 3, 3)) if small else _table(tt, r)
    idx, off = _batch(table.num_rows, nnz, bags, nnz + bags)
    out = torch.full((bags, 128), float("nan"), device="cuda")
    tt.tt_emb_bag_forward_static(table, idx, off, out)
    plan = tt.tt_index_reorder(table, idx, off)
    assert torch.equal(out, tt.tt_emb_bag_forward(table, plan, idx, off))


@pytest.mark.parametrize("r", [32, 64])
@pytest.mark.parametrize("nnz", [0, 20])
def test_many_bags_cost_no_more_than_with_a_plan(r, nnz):
    """Measured 8 us against 13 (no lookups: one workgroup's plan) and 35."""
    import paper_2507_14668_amd as tt
    print("case direct cost r=%d nnz=%d" % (r, nnz), flush=True)
    table, bags = _table(tt, r), 16384
    idx, off = _batch(table.num_rows, nnz, bags, 3)
    out = torch.empty((bags, 128), device="cuda")
    ws = tt.alloc_workspace(table, nnz, bags)

    def took(call):
        each = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(100):
                call()
            b.record()
            b.synchronize()
            each.append(a.elapsed_time(b))
        return min(each)

    static = took(lambda: tt.tt_emb_bag_forward_static(table, idx, off, out))
    planned = took(lambda: tt.tt_emb_bag_forward(table, tt.tt_index_reorder(table, idx, off, workspace=ws), idx, off, out=out))
    assert static <= planned, (static, planned)


@pytest.mark.parametrize("nnz", [20, 200])
def test_malformed_offsets_and_a_table_smaller_than_the_batch(nnz):
    import paper_2507_14668_amd as tt
    print("case direct malformed nnz=%d" % nnz, flush=True)
    table = _table(tt, 32)
    idx, off = _batch(table.num_rows, nnz, 6, 5)
    off[2], off[4] = nnz + 9, -3  # not monotone, outside of the batch
    small = _table(tt, 64, rows=17, n=(2, 3, 3))
    sidx = torch.randint(0, 17, (nnz,), device="cuda")
    for t, i, o in ((table, idx, off), (small, sidx, torch.tensor([0, 5, nnz], device="cuda"))):
        out = torch.full((o.numel() - 1, 128), float("nan"), device="cuda")
        tt.tt_emb_bag_forward_static(t, i, o, out)
        plan = tt.tt_index_reorder(t, i, o)
        assert torch.equal(out, tt.tt_emb_bag_forward(t, plan, i, o))


def test_replayed_from_a_graph():
    import paper_2507_14668_amd as tt
    print("case direct graph", flush=True)
    table = _table(tt, 32)
    for nnz, bags in ((20, 2), (700, 90)):
        idx, off = _batch(table.num_rows, nnz, bags, 1)
        out = torch.zeros(bags, 128, device="cuda")
        tt.tt_emb_bag_forward_static(table, idx, off, out)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            tt.tt_emb_bag_forward_static(table, idx, off, out, stream=torch.cuda.current_stream())
        for turn in range(3):
            idx.copy_(_batch(table.num_rows, nnz, bags, turn)[0])
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            plan = tt.tt_index_reorder(table, idx, off)
            assert torch.equal(out, tt.tt_emb_bag_forward(table, plan, idx, off))


@pytest.mark.parametrize("r,nnz,bags", [
    (r, nnz, bags) for r, top in ((32, 40000), (64, 12000))
    for nnz, bags in ((1, 1), (20, 1), (65, 3), (300, 1), (700, 90), (2048, 300), (2049, 300), (top, top // 10), (2 * top, top // 10), (50, 30000))])
def test_bf16_inference_without_a_plan(r, nnz, bags):
    """On both sides of the rule the module gives what the planned call gives, to the fp32 rounding of sums over the bag's
    lookups (chains of R products and of the lookups, added in another order: a few 1e-7 of the largest output)."""
    import paper_2507_14668_amd as tt
    from paper_2507_14668_amd import binding
    print("case direct bf16 r=%d nnz=%d bags=%d" % (r, nnz, bags), flush=True)
    n, d = (60, 50, 40), (4, 8, 4)
    bag = tt.TTEmbeddingBag(n[0] * n[1] * n[2] - 7, 128, n=n, d=d, ranks=(r, r), include_last_offset=True,
                            generator=torch.Generator(device="cuda").manual_seed(r)).bf16_inference()
    table = bag._table(bag.cores())
    idx, off = _batch(table.num_rows, nnz, bags, nnz + bags)
    plan = tt.tt_index_reorder(table, idx, off)
    ref = tt.tt_emb_bag_forward_bf16(table, bag._bf16_cores, plan, off)
    direct = binding.tt_emb_bag_forward_bf16_direct(table, bag._bf16_cores, idx, off)
    for out in (bag.forward_bf16(idx, off), direct):
        assert (out - ref).abs().max() <= 3e-6 * ref.abs().max() and (out - ref).norm() <= 1e-6 * ref.norm()
    if not binding.tt_forward_bf16_direct_pays(table, nnz, bags):
        assert torch.equal(bag.forward_bf16(idx, off), ref)
