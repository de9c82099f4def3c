"""The library's HIP kernels and host code compiled for the CPU (tests/cpu_emulation) and

  * compared with the oracle through the same C ABI (forward, backward, update, fused update, plan
    arrays, both arms) -- the kernels' logic is checked here without a GPU;
  * run under AddressSanitizer + UBSan, single-table and batched, on seeded inputs: any
    out-of-bounds or misaligned access of a kernel fails the test.  The batched entry points, which
    are switched off in the GPU build, are switched on in this build.

Nothing here stands in for the GPU parity tests: the emulation runs one workgroup at a time and
knows nothing about the hardware's memory system."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

import tt_workloads as wl

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "cpu_emulation"))
import build as emu_build  # noqa: E402

BUILD_DIR = os.path.join(os.path.dirname(os.path.abspath(__file__)), "cpu_emulation", "_build")
pytestmark = pytest.mark.skipif(not emu_build.available(), reason="host clang++ of the ROCm toolchain not found")


@pytest.fixture(scope="module")
def emu():
    return _load(emu_build.build_shared(BUILD_DIR))


def _load(path):
    from paper_2507_14668_amd import binding
    lib = ctypes.CDLL(path)
    vp, i64, f32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_float
    lib.tt_workspace_bytes.restype = ctypes.c_size_t
    lib.tt_workspace_bytes.argtypes = [vp, i64, i64]
    lib.tt_index_reorder.argtypes = [vp, vp, vp, i64, i64, vp, vp, ctypes.c_size_t, vp, vp]
    lib.tt_emb_bag_forward.argtypes = [vp, vp, vp, vp, i64, i64, vp, vp]
    lib.tt_emb_bag_backward.argtypes = [vp, vp, vp, vp, i64, i64, vp, vp, vp]
    lib.tt_core_sgd_update.argtypes = [vp, vp, vp, f32, vp]
    lib.tt_emb_bag_backward_sgd.argtypes = [vp, vp, vp, vp, i64, i64, vp, f32, vp]
    return lib, binding


def _ptr(a):
    return ctypes.c_void_p(a.ctypes.data)


def _aligned(nbytes):
    # all ones (NaN as a float): a block that an earlier call has freed would still hold the right results, and a kernel that
    # writes nothing would pass
    raw = np.full(nbytes + 256, 0xFF, dtype=np.uint8)
    off = (-raw.ctypes.data) % 256
    return raw[off:off + nbytes]


def _table(binding, shape, cores):
    t = binding.CTable()
    t.num_rows = shape.num_rows
    t.n[:], t.d[:], t.r[:] = shape.n, shape.d, shape.r
    for k in range(3):
        t.core[k] = cores[k].ctypes.data
    return t


def _run(emu, shape, cores, idx, off, grad, lr):
    lib, binding = emu
    cores = [np.ascontiguousarray(c, dtype=np.float32).copy() for c in cores]
    idx, off = np.ascontiguousarray(idx, dtype=np.int64), np.ascontiguousarray(off, dtype=np.int64)
    grad = np.ascontiguousarray(grad, dtype=np.float32)
    nnz, nb = len(idx), len(off) - 1
    table = _table(binding, shape, cores)
    ws = _aligned(lib.tt_workspace_bytes(ctypes.byref(table), nnz, nb))
    plan = binding.CPlan()
    assert lib.tt_index_reorder(ctypes.byref(table), _ptr(idx), _ptr(off), nnz, nb, None, _ptr(ws), ws.nbytes,
                                ctypes.byref(plan), None) == 0
    res = {}

    def ints(name, count):
        o = getattr(plan, name) - ws.ctypes.data
        return ws[o:o + 4 * count].view(np.int32).copy()

    counts = ints("counts", 16)
    ur, up = int(counts[0]), int(counts[1])
    res["plan_arrays"] = dict(U_r=ur, U_p=up, num_valid=int(counts[2]), status=int(counts[4]), uniq_row=ints("uniq_row", ur),
                       row_seg=ints("row_seg", ur + 1), uniq_pref=ints("uniq_pref", up), pref_seg=ints("pref_seg", up + 1),
                       lookup2row=ints("lookup2row", nnz), i2_seg=ints("i2_seg", shape.n[1] + 1),
                       i3_seg=ints("i3_seg", shape.n[2] + 1), i1_seg=ints("i1_seg", shape.n[0] + 1))
    for arm, pl in (("plan", ctypes.byref(plan)), ("naive", None)):
        out = np.full((nb, shape.dim), np.nan, dtype=np.float32)
        assert lib.tt_emb_bag_forward(ctypes.byref(table), pl, _ptr(idx), _ptr(off), nnz, nb, _ptr(out), None) == 0
        dg = [np.full_like(c, np.nan) for c in cores]
        arr = (ctypes.c_void_p * 3)(*[g.ctypes.data for g in dg])
        assert lib.tt_emb_bag_backward(ctypes.byref(table), pl, _ptr(idx), _ptr(off), nnz, nb, _ptr(grad), arr, None) == 0
        res[arm] = (out, dg)
    # update (touched slices) after the planned backward, and the fused call on fresh cores
    dg = res["plan"][1]
    arr = (ctypes.c_void_p * 3)(*[g.ctypes.data for g in dg])
    upd = [c.copy() for c in cores]
    t_upd = _table(binding, shape, upd)
    assert lib.tt_core_sgd_update(ctypes.byref(t_upd), ctypes.byref(plan), arr, ctypes.c_float(lr), None) == 0
    fused = [c.copy() for c in cores]
    t_fused = _table(binding, shape, fused)
    assert lib.tt_emb_bag_backward_sgd(ctypes.byref(t_fused), ctypes.byref(plan), _ptr(idx), _ptr(off), nnz, nb,
                                       _ptr(grad), ctypes.c_float(lr), None) == 0
    res["updated"], res["fused"] = upd, fused
    return res


@pytest.mark.parametrize("name,n,d,r,nb,ml", [
    ("plain", (5, 4, 6), (2, 3, 2), (1, 3, 5, 1), 150, 6),
    ("mfma_r32_split", (9, 3, 5), (4, 8, 4), (1, 32, 32, 1), 260, 5),   # 3 core-1 slices: split workgroups
    ("mfma_r64_two_strips", (3, 2, 11), (4, 8, 4), (1, 64, 64, 1), 120, 4),
    # rows looked up hundreds of times: segments of the gradient merge that span whole workgroups of stage 1
    ("mfma_r64_hot_rows", (2, 1, 2), (4, 8, 4), (1, 64, 64, 1), 800, 4),
    ("plain_hot_rows", (1, 2, 2), (2, 3, 2), (1, 3, 5, 1), 2500, 3),
    # more than 64 prefixes under one i2 (the staged plan entries are refilled) and prefixes with more
    # than 32 distinct rows (row batches that cut a prefix's rows at any position)
    ("mfma_r32_refill", (75, 1, 3), (4, 8, 4), (1, 32, 32, 1), 400, 3),
    ("mfma_r64_row_batches", (2, 2, 45), (4, 8, 4), (1, 64, 64, 1), 300, 4),
    # row factors above 1023: the groupings by i2 / i3 become radix sorts of more than one digit
    ("mfma_r32_wide_n2", (1, 2100, 2), (4, 8, 4), (1, 32, 32, 1), 200, 3),
    ("plain_wide_n3", (2, 1, 1500), (2, 3, 2), (1, 3, 5, 1), 300, 3),
    # 31-bit row keys (2.1e9 rows): four radix passes
    ("plain_31_bit_keys", (1290, 1290, 1290), (2, 3, 2), (1, 3, 5, 1), 300, 4),
])
def test_emulated_kernels_match_oracle(emu, ora, name, n, d, r, nb, ml):
    import gpu_util as g
    shape, cores, idx, off, grad = wl.small_random_problem(301, n=n, d=d, r=r, num_bags=nb, max_len=ml, sigma=0.2)
    lr = 0.05
    res = _run(emu, shape, cores, idx, off, grad, lr)
    ref_plan = ora.reorder_plan(shape, idx, off)
    p = res["plan_arrays"]
    assert p["status"] == 0 and p["num_valid"] == ref_plan["num_valid"]
    for key in ("uniq_row", "row_seg", "uniq_pref", "pref_seg", "lookup2row"):
        assert np.array_equal(p[key], ref_plan[key]), key
    i3 = np.sort(ref_plan["uniq_row"] % shape.n[2])
    assert np.array_equal(p["i3_seg"], np.searchsorted(i3, np.arange(shape.n[2] + 1)))
    i2 = np.sort(ref_plan["uniq_pref"] % shape.n[1])
    assert np.array_equal(p["i2_seg"], np.searchsorted(i2, np.arange(shape.n[1] + 1)))
    assert np.array_equal(p["i1_seg"], np.searchsorted(ref_plan["uniq_pref"] // shape.n[1], np.arange(shape.n[0] + 1)))
    ref_out = ora.forward(shape, cores, idx, off)
    ref_dg = ora.backward(shape, cores, idx, off, grad)
    for arm in ("plan", "naive"):
        out, dg = res[arm]
        g.assert_close_rows(out, ref_out, g.FWD_RTOL, shape.dim, "%s forward (%s)" % (name, arm))
        g.assert_grads_close(shape, dg, ref_dg, what="%s dG (%s)" % (name, arm))
    g.assert_grads_close(shape, res["updated"], ora.sgd(cores, ref_dg, lr), what="%s updated G" % name)
    for k in range(3):
        assert np.array_equal(res["fused"][k], res["updated"][k]), "fused update differs from backward + update"


def test_emulated_one_hot_batch_and_mixed_bag_lengths(emu, ora):
    """One lookup per bag (the bag sum takes four bags of a lane group at a time) and a batch whose bags
    hold zero or one lookup (the fast path gives way to the general one wherever a bag is not single)."""
    import gpu_util as g
    shape, cores, _, _, _ = wl.small_random_problem(41, n=(5, 4, 6), d=(2, 3, 2), r=(1, 3, 5, 1))
    rng = np.random.default_rng(5)
    sparse = np.zeros(4000, np.int64)  # runs of more than a tile's worth of empty bags between the lookups
    sparse[[0, 1500, 1501, 3999]] = (3, 2, 1200, 4)
    for nb, lens in ((1500, None), (1100, rng.integers(0, 2, 1100)), (4000, sparse)):
        lens = np.ones(nb, np.int64) if lens is None else lens
        off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        idx = rng.integers(0, shape.num_rows, int(off[-1])).astype(np.int64)
        grad = rng.standard_normal(nb * shape.dim).astype(np.float32)
        res = _run(emu, shape, cores, idx, off, grad, 0.05)
        ref_out = ora.forward(shape, cores, idx, off)
        assert np.array_equal(res["plan_arrays"]["lookup2row"], ora.reorder_plan(shape, idx, off)["lookup2row"])
        for arm in ("plan", "naive"):
            g.assert_close_rows(res[arm][0], ref_out, g.FWD_RTOL, shape.dim, "one-hot forward (%s)" % arm)
        g.assert_grads_close(shape, res["plan"][1], ora.backward(shape, cores, idx, off, grad), what="one-hot dG")


@pytest.mark.parametrize("nb,ml,rows,hot,max_group", [(300, 9, 400, 5, 64), (40, 300, 3000, 0, 16), (200, 5, 50, 45, 64)])
def test_emulated_index_graph_edges_match_oracle(emu, ora, nb, ml, rows, hot, max_group):
    """The edge-generation job (pairs per bag, two stable radix sorts, run heads) against the loop oracle:
    short bags, bags longer than a wavefront round and than the per-bag cap, almost every row hot."""
    lib, _ = emu
    rng = np.random.default_rng(nb)
    lens = rng.integers(0, ml + 1, nb)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = np.minimum((rows ** rng.random(int(off[-1]))).astype(np.int64), rows - 1)  # skewed
    idx[::17] = -1
    rank = rng.permutation(rows).astype(np.int32)
    ref = ora.index_graph_edges(idx, off, rank, hot, max_group)
    cap = max(1, int(sum(min(l, max_group) * (min(l, max_group) - 1) // 2 for l in lens)))
    lib.tt_index_graph_workspace_bytes.restype = ctypes.c_size_t
    lib.tt_index_graph_workspace_bytes.argtypes = [ctypes.c_int64, ctypes.c_int64]
    ws = _aligned(lib.tt_index_graph_workspace_bytes(nb, cap))
    eu, ev, ew = (np.full(cap, -1, np.int32) for _ in range(3))
    counts = np.zeros(4, np.int32)
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    lib.tt_index_graph_edges.argtypes = [vp, vp, i64, i64, vp, i64, i64, ctypes.c_int32, vp, ctypes.c_size_t, i64,
                                         vp, vp, vp, vp, vp]
    assert lib.tt_index_graph_edges(_ptr(idx), _ptr(off), len(idx), nb, _ptr(rank), rows, hot, max_group, _ptr(ws),
                                    ws.nbytes, cap, _ptr(eu), _ptr(ev), _ptr(ew), _ptr(counts), None) == 0
    assert counts[2] == 0 and counts[0] == sum(ref.values()) and counts[1] == len(ref)
    got = {(int(u), int(v)): int(w) for u, v, w in zip(eu[:counts[1]], ev[:counts[1]], ew[:counts[1]])}
    assert got == ref
    keys = list(zip(eu[:counts[1]].tolist(), ev[:counts[1]].tolist()))
    assert keys == sorted(keys), "edges must come out sorted by (u, v)"
    # a capacity that is too small is reported, and nothing is produced
    if sum(ref.values()) > 1:
        assert lib.tt_index_graph_edges(_ptr(idx), _ptr(off), len(idx), nb, _ptr(rank), rows, hot, max_group, _ptr(ws),
                                        ws.nbytes, sum(ref.values()) - 1, _ptr(eu), _ptr(ev), _ptr(ew), _ptr(counts), None) == 0
        assert counts[2] == 1 and counts[1] == 0


@pytest.fixture(scope="module")
def asan_harness():
    return emu_build.build_harness(BUILD_DIR, "address")


@pytest.mark.parametrize("kind,shuffle", [("mfma", None), ("plain", None), ("unaligned", None), ("wide", None), ("keys31", None),
                                          ("mfma", "11"), ("plain", "12")])
def test_sanitized_single_and_batched_calls(asan_harness, kind, shuffle):
    """Every entry point under AddressSanitizer + UBSan.  While a launch runs, the host structs of the
    C ABI (tables, plans, batch items) and the library's host copies of the table descriptors are
    poisoned: a kernel that followed a host pointer -- harmless on the CPU, a fault on a GPU -- is
    reported.  With `shuffle` the workgroups of every launch run in a seeded random order over both grid
    dimensions, so that the tables of a batched launch are interleaved."""
    env = dict(os.environ, ASAN_OPTIONS="detect_stack_use_after_return=0:detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1")
    if shuffle:
        env["EMU_SHUFFLE"] = shuffle
    # the kinds with very wide tables run the planned arm only: a dense update sweep over their cores
    # takes the emulation minutes and is no other code than on the small tables
    planned_only = kind in ("wide", "keys31")
    res = subprocess.run([asan_harness, kind] + (["1"] if planned_only else []), capture_output=True, text=True, env=env,
                         timeout=600)
    text = res.stdout + res.stderr
    assert res.returncode == 0, text[-4000:]
    assert "ERROR" not in text and "runtime error" not in text, text[-4000:]
    assert text.count("identical") == (1 if planned_only else 2), text[-2000:]  # per arm: batched == single-table
    assert ", 0 values off" in text, text[-2000:]  # the same tables as one fused table: same results to rounding


def test_emulated_kernels_on_random_shapes(emu, ora):
    """Seeded random shapes within the library's limits (ranks and factors that are not powers of
    two, single-slice cores, padded row counts, the matrix-core shapes): every arm against the
    oracle, and the fused update bit for bit against backward + update."""
    import gpu_util as g
    rng = np.random.default_rng(20250714)
    for case in range(14):
        while True:
            n = tuple(int(x) for x in rng.integers(1, 9, size=3))
            d = tuple(int(x) for x in rng.choice([1, 2, 3, 4, 5, 8], size=3))
            r1, r2 = int(rng.choice([1, 2, 3, 7, 16, 33, 64])), int(rng.choice([1, 2, 5, 8, 17, 32, 64]))
            if rng.random() < 0.25:
                d, r1 = (4, 8, 4), int(rng.choice([32, 64]))
                r2 = r1
            dim, p12, s2 = d[0] * d[1] * d[2], d[0] * d[1] * r2, d[1] * r2
            lds = d[0] * r1 + d[0] * d[1] * (r2 | 1) + p12 + dim + 8 * r2 * d[2]
            if dim <= 1024 and p12 <= 4096 and s2 <= 4096 and lds * 4 <= 65536:
                break
        cap = n[0] * n[1] * n[2]
        num_rows = int(rng.integers(max(1, cap - n[2] + 1), cap + 1))
        nb, ml = int(rng.integers(1, 100)), int(rng.integers(1, 8))
        shape, cores, idx, off, grad = wl.small_random_problem(7000 + case, n=n, d=d, r=(1, r1, r2, 1), num_rows=num_rows,
                                                              num_bags=nb, max_len=ml, sigma=0.3)
        what = "n=%s d=%s r=(%d,%d) rows=%d" % (n, d, r1, r2, num_rows)
        res = _run(emu, shape, cores, idx, off, grad, 0.05)
        ref_out, ref_dg = ora.forward(shape, cores, idx, off), ora.backward(shape, cores, idx, off, grad)
        for arm in ("plan", "naive"):
            out, dg = res[arm]
            g.assert_close_rows(out, ref_out, g.FWD_RTOL, shape.dim, "%s forward (%s)" % (what, arm))
            g.assert_grads_close(shape, dg, ref_dg, what="%s dG (%s)" % (what, arm))
        for k in range(3):
            assert np.array_equal(res["fused"][k], res["updated"][k]), what


def test_results_do_not_depend_on_workgroup_order(asan_harness):
    """The emulation runs the workgroups of a launch one after the other; last to first must give
    the same bits as first to last (no kernel relies on another workgroup of its launch)."""
    sums = []
    for reverse in (False, True):
        env = dict(os.environ, ASAN_OPTIONS="detect_stack_use_after_return=0:detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1")
        if reverse:
            env["EMU_REVERSE"] = "1"
        res = subprocess.run([asan_harness, "mfma"], capture_output=True, text=True, env=env, timeout=900)
        text = res.stdout + res.stderr
        assert res.returncode == 0 and "ERROR" not in text, text[-3000:]
        sums.append([ln for ln in text.splitlines() if ln.startswith("checksum")])
    # first checksum: the planned arm (no atomics, must not move); second: the naive arm, whose
    # backward adds with float atomics in arrival order and is not expected to be bit-stable
    assert len(sums[0]) == 2 and sums[0][0] == sums[1][0]


def test_pair_walk_of_the_core1_reduction():
    """The chunks of (prefix, j1) pairs that the core-1 gradient of the plain kernels is summed over: the walk names
    every pair once and in order, also where there are 2^31 pairs and more (two million prefixes, d1 = 1023)."""
    res = subprocess.run([emu_build.build_unit(BUILD_DIR, "pair_walk")], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr


def test_launches_of_tables_with_millions_of_slices(emu):
    """2.2 million i1 and vectors of two widths (d3 = 3 beside ranks of four): one workgroup per slice and column part would
    be more threads than a launch holds, so the core-2 and core-0 sums take the two-stage route; the fused update of
    the touched slices against 64 bits, every other slice of core 0 unchanged."""
    lib, binding = emu
    n, d, r = (2_200_000, 2, 2), (4, 2, 3), (1, 16, 5, 1)
    rng = np.random.default_rng(9)
    idx = np.concatenate([rng.integers(0, 4 * n[0], 20), [0, 4 * n[0] - 1, 3, 3]]).astype(np.int64)
    u, inv = np.unique(idx, return_inverse=True)
    off = np.arange(len(idx) + 1, dtype=np.int64)
    i3, i2, i1 = u % 2, u // 2 % 2, u // 4
    cores = [np.zeros(n[0] * d[0] * r[1], np.float32)] + [rng.standard_normal(s).astype(np.float32) for s in
                                                          (r[1] * n[1] * d[1] * r[2], r[2] * n[2] * d[2])]
    g1 = cores[0].reshape(n[0], d[0], r[1])
    touched = np.unique(i1)
    g1[touched] = rng.standard_normal((len(touched), d[0], r[1]))
    old = [g1[touched].astype(np.float64)] + [c.astype(np.float64) for c in cores[1:]]
    grad = rng.standard_normal((len(idx), d[0], d[1], d[2])).astype(np.float32)
    shape = wl.TableShape(4 * n[0], n, d, r)
    table = _table(binding, shape, cores)
    ws, plan = _aligned(lib.tt_workspace_bytes(ctypes.byref(table), len(idx), len(idx))), binding.CPlan()
    assert lib.tt_index_reorder(ctypes.byref(table), _ptr(idx), _ptr(off), len(idx), len(idx), None, _ptr(ws), ws.nbytes,
                                ctypes.byref(plan), None) == 0
    assert lib.tt_emb_bag_backward_sgd(ctypes.byref(table), ctypes.byref(plan), _ptr(idx), _ptr(off), len(idx), len(idx),
                                       _ptr(grad), ctypes.c_float(0.25), None) == 0
    merged = np.zeros((len(u),) + d)
    np.add.at(merged, inv, grad.astype(np.float64))
    a = old[0][np.searchsorted(touched, i1)]
    b = old[1].reshape(r[1], n[1], d[1], r[2])[:, i2].transpose(1, 0, 2, 3)
    c = old[2].reshape(r[2], n[2], d[2])[:, i3].transpose(1, 0, 2)
    h = np.einsum("uabc,usc->uabs", merged, c)
    new = [old[0].copy(), old[1].reshape(r[1], n[1], d[1], r[2]).copy(), old[2].reshape(r[2], n[2], d[2]).copy()]
    for k in range(len(u)):
        new[0][np.searchsorted(touched, i1[k])] -= 0.25 * np.einsum("abs,rbs->ar", h[k], b[k])
        new[1][:, i2[k]] -= 0.25 * np.einsum("ar,abs->rbs", a[k], h[k])
        new[2][:, i3[k]] -= 0.25 * np.einsum("ar,rbs,abc->sc", a[k], b[k], merged[k])
    for got, ref in ((g1[touched], new[0]), (cores[1].reshape(new[1].shape), new[1]), (cores[2].reshape(new[2].shape), new[2])):
        assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
    assert np.count_nonzero(g1.any(axis=(1, 2))) == len(touched)


@pytest.mark.parametrize("lookups,shuffle", [(9000, None), (9000, "21"), (70000, None)])
def test_sanitized_plans_of_long_batches(asan_harness, lookups, shuffle):
    """The plan built by several launches, under AddressSanitizer + UBSan and against a host construction, bit for bit: ten
    sort tiles and (70 000 lookups) more than 64, where groups of tiles are counted; two to four radix passes; row factors
    above 1023; malformed offsets; and batched calls that mix such tables with short ones, one lookup and no lookups."""
    env = dict(os.environ, ASAN_OPTIONS="detect_stack_use_after_return=0:detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1")
    if shuffle:
        env["EMU_SHUFFLE"] = shuffle
    res = subprocess.run([asan_harness, "plans", str(lookups)], capture_output=True, text=True, env=env, timeout=600)
    text = res.stdout + res.stderr
    assert res.returncode == 0 and "plans: all right" in text, text[-4000:]
    assert "ERROR" not in text and "runtime error" not in text, text[-4000:]


@pytest.mark.parametrize("nnz,bags,n,threads", [
    (20, 1, (200, 250, 200), 64), (32, 64, (256, 256, 256), 64), (33, 64, (256, 256, 256), 256), (32, 65, (256, 256, 256), 256),
    (32, 64, (257, 3, 4), 256), (32, 64, (3, 257, 4), 256), (32, 64, (3, 4, 257), 256), (60, 1000, (16000, 3, 2), 256),
    (256, 300, (7, 9, 11), 256), (257, 300, (7, 9, 11), 512)])
def test_who_builds_a_short_plan(emu, ora, capfd, monkeypatch, nnz, bags, n, threads):
    """Only the shortest batches of small tables get their plan from a single wavefront, which walks the bags and the
    segment starts alone; the plan is the oracle's on both sides of every limit."""
    rng = np.random.default_rng(nnz + bags)
    shape, cores, _, _, _ = wl.small_random_problem(3, n=n, d=(1, 2, 2), r=(1, 1, 2, 1))
    off = np.concatenate([[0], np.sort(rng.integers(0, nnz + 1, bags - 1)), [nnz]]).astype(np.int64)
    idx = rng.integers(0, shape.num_rows, nnz).astype(np.int64)
    monkeypatch.setenv("EMU_TRACE", "1")
    res = _run(emu, shape, cores, idx, off, rng.standard_normal(bags * 4), 0.05)["plan_arrays"]
    launches = [ln for ln in capfd.readouterr().err.splitlines() if "k_plan_small" in ln]
    assert len(launches) == 1 and " block %d " % threads in launches[0], launches
    ref = ora.reorder_plan(shape, idx, off)
    for key in ("uniq_row", "row_seg", "uniq_pref", "pref_seg", "lookup2row"):
        assert np.array_equal(res[key], ref[key]), key
    i3, i2 = np.sort(ref["uniq_row"] % n[2]), np.sort(ref["uniq_pref"] % n[1])
    assert np.array_equal(res["i3_seg"], np.searchsorted(i3, np.arange(n[2] + 1)))
    assert np.array_equal(res["i2_seg"], np.searchsorted(i2, np.arange(n[1] + 1)))
    assert np.array_equal(res["i1_seg"], np.searchsorted(ref["uniq_pref"] // n[1], np.arange(n[0] + 1)))


def _exact_grads(shape, cores, idx, off, grad):
    """Core gradients of the batch in 64 bits, in the layout of the cores."""
    n, d, (_, r1, r2, _) = shape.n, shape.d, shape.r
    a, b, c = (x.astype(np.float64) for x in cores)
    a, b, c = a.reshape(n[0], d[0], r1), b.reshape(r1, n[1], d[1], r2), c.reshape(r2, n[2], d[2])
    u, inv = np.unique(idx, return_inverse=True)
    g = np.zeros((len(u),) + tuple(d))
    np.add.at(g, inv, grad.astype(np.float64).reshape((-1,) + tuple(d))[np.repeat(np.arange(len(off) - 1), np.diff(off))])
    i1, i2, i3 = u // n[2] // n[1], u // n[2] % n[1], u % n[2]
    au, bu, cu = a[i1], b[:, i2].transpose(1, 0, 2, 3), c[:, i3].transpose(1, 0, 2)
    p12 = np.einsum("uar,urbs->uabs", au, bu, optimize=True)
    h = np.einsum("uabc,usc->uabs", g, cu, optimize=True)
    dg = [np.zeros_like(a), np.zeros((n[1], r1, d[1], r2)), np.zeros((n[2], r2, d[2]))]
    np.add.at(dg[0], i1, np.einsum("uabs,urbs->uar", h, bu, optimize=True))
    np.add.at(dg[1], i2, np.einsum("uar,uabs->urbs", au, h, optimize=True))
    np.add.at(dg[2], i3, np.einsum("uabs,uabc->usc", p12, g, optimize=True))
    return dg[0].ravel(), dg[1].transpose(1, 0, 2, 3).ravel(), dg[2].transpose(1, 0, 2).ravel()


# largest geometric mean over eight batches of the relative error (2-norm) of the three core gradients: what the kernels
# with a workgroup per prefix and two-stage sums show on the same batches (emulated sums are the same on every machine)
@pytest.mark.parametrize("n,d,r,bags,limits", [
    ((20, 21, 20), (2, 4, 6), (1, 12, 20, 1), 700, (1.127e-7, 1.315e-7, 1.163e-7)),  # one sum's vectors are fours, the other's are not
    ((20, 20, 20), (2, 4, 6), (1, 8, 8, 1), 700, (1.157e-7, 1.308e-7, 1.100e-7)),
    ((30, 30, 30), (4, 4, 4), (1, 16, 16, 1), 700, (1.295e-7, 1.909e-7, 1.534e-7)),
    ((10, 10, 10), (2, 2, 4), (1, 4, 4, 1), 400, (1.152e-7, 1.069e-7, 1.543e-7)),
])
def test_order_of_additions_costs_no_precision(emu, n, d, r, bags, limits):
    """Core gradients of the plain kernels against 64 bits: the order in which products, rows and slices are added may
    change, their error may not grow."""
    lib, binding = emu
    logs = np.zeros(3)
    for seed in range(8):
        shape, cores, idx, off, grad = wl.small_random_problem(900 + seed, n=n, d=d, r=r, num_bags=bags, max_len=5, sigma=0.3)
        table = _table(binding, shape, cores)
        ws, plan = _aligned(lib.tt_workspace_bytes(ctypes.byref(table), len(idx), bags)), binding.CPlan()
        assert lib.tt_index_reorder(ctypes.byref(table), _ptr(idx), _ptr(off), len(idx), bags, None, _ptr(ws), ws.nbytes,
                                    ctypes.byref(plan), None) == 0
        dg = [_aligned(c.nbytes).view(np.float32) for c in cores]
        arr = (ctypes.c_void_p * 3)(*[g.ctypes.data for g in dg])
        grad = np.ascontiguousarray(grad, np.float32)
        assert lib.tt_emb_bag_backward(ctypes.byref(table), ctypes.byref(plan), _ptr(idx), _ptr(off), len(idx), bags, _ptr(grad), arr, None) == 0
        logs += [np.log(np.linalg.norm(got - ref) / np.linalg.norm(ref)) for got, ref in zip(dg, _exact_grads(shape, cores, idx, off, grad))]
    errors = np.exp(logs / 8)
    assert np.all(errors <= np.array(limits)), (errors, limits)


@pytest.mark.parametrize("case", ["one_hot", "zero_or_one", "empty_runs", "one_bag"])
def test_emulated_bag_search_of_long_batches(emu, ora, case):
    """The bag of every lookup in batches of several sort tiles: one lookup per bag (no search), bags of zero or one, runs
    of thousands of empty bags (beyond the window of offsets that a tile stages), one bag over all tiles."""
    lib, binding = emu
    rng = np.random.default_rng(6)
    lens = {"one_hot": np.ones(2500, np.int64), "zero_or_one": rng.integers(0, 2, 5200), "empty_runs": np.zeros(9000, np.int64),
            "one_bag": np.array([0, 3100, 0])}[case]
    if case == "empty_runs":
        lens[[0, 3000, 3001, 8999]] = (700, 900, 500, 1300)
    shape, cores, _, _, _ = wl.small_random_problem(42, n=(5, 4, 6), d=(1, 1, 2), r=(1, 1, 1, 1))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = rng.integers(-1, shape.num_rows + 1, int(off[-1])).astype(np.int64)
    table, plan = _table(binding, shape, cores), binding.CPlan()
    ws = _aligned(lib.tt_workspace_bytes(ctypes.byref(table), len(idx), len(lens)))
    assert len(idx) > 2048
    assert lib.tt_index_reorder(ctypes.byref(table), _ptr(idx), _ptr(off), len(idx), len(lens), None, _ptr(ws), ws.nbytes,
                                ctypes.byref(plan), None) == 0
    ref = ora.reorder_plan(shape, idx, off)

    def ints(name, count):
        o = getattr(plan, name) - ws.ctypes.data
        return ws[o:o + 4 * count].view(np.int32)
    assert int(ints("counts", 5)[4]) == 1  # lookups outside the table, valid offsets
    for key in ("bag_of_sorted", "perm", "sorted_row"):
        assert np.array_equal(ints(key, ref["num_valid"]), ref[key]), key
    assert np.array_equal(ints("lookup2row", len(idx)), ref["lookup2row"])


def _backward_with_trace(emu, capfd, monkeypatch, n, d, r, nnz, seed=5):
    """(launch lines, gradients, exact gradients) of one planned backward of `nnz` one-lookup bags."""
    lib, binding = emu
    rng = np.random.default_rng(seed)
    shape, cores, _, _, _ = wl.small_random_problem(seed, n=n, d=d, r=r, num_bags=1, max_len=1, sigma=0.3)
    idx, off = rng.integers(0, shape.num_rows, nnz).astype(np.int64), np.arange(nnz + 1, dtype=np.int64)
    grad = rng.standard_normal(nnz * shape.dim).astype(np.float32)
    table, plan = _table(binding, shape, cores), binding.CPlan()
    ws = _aligned(lib.tt_workspace_bytes(ctypes.byref(table), nnz, nnz))
    assert lib.tt_index_reorder(ctypes.byref(table), _ptr(idx), _ptr(off), nnz, nnz, None, _ptr(ws), ws.nbytes, ctypes.byref(plan), None) == 0
    dg = [_aligned(c.nbytes).view(np.float32) for c in cores]
    for x in dg:
        x.fill(np.nan)
    arr = (ctypes.c_void_p * 3)(*[x.ctypes.data for x in dg])
    monkeypatch.setenv("EMU_TRACE", "1")
    capfd.readouterr()
    assert lib.tt_emb_bag_backward(ctypes.byref(table), ctypes.byref(plan), _ptr(idx), _ptr(off), nnz, nnz, _ptr(grad), arr, None) == 0
    launches, ref, old = capfd.readouterr().err.splitlines(), _exact_grads(shape, cores, idx, off, grad), [c.copy() for c in cores]
    assert lib.tt_emb_bag_backward_sgd(ctypes.byref(table), ctypes.byref(plan), _ptr(idx), _ptr(off), nnz, nnz, _ptr(grad),
                                       ctypes.c_float(0.5), None) == 0
    for new, before, x in zip(cores, old, dg):  # the fused update takes the same routes
        assert np.array_equal(new, (before - 0.5 * x.astype(np.float64)).astype(np.float32))
    return launches, dg, ref


@pytest.mark.parametrize("n,d,r,nnz,whole", [
    ((50, 50, 2), (2, 2, 3), (1, 16, 5, 1), 2049, True), ((50, 50, 2), (2, 2, 3), (1, 16, 5, 1), 2050, False),  # rows per i3
    ((34, 33, 16), (2, 2, 3), (1, 16, 5, 1), 16416, True),
    ((1, 2500, 9), (2, 2, 3), (1, 16, 5, 1), 2048, True), ((1, 2500, 9), (2, 2, 3), (1, 16, 5, 1), 2049, False),  # prefixes per i1
    ((2047, 2, 2), (2, 2, 3), (1, 16, 5, 1), 60, True), ((2048, 2, 2), (2, 2, 3), (1, 16, 5, 1), 60, False),  # slices
    ((50, 50, 2), (2, 2, 4), (1, 16, 5, 1), 2050, True), ((2048, 2, 2), (2, 2, 4), (1, 16, 5, 1), 60, True),  # vectors of one width
])
def test_who_sums_the_core2_and_core0_gradients(emu, capfd, monkeypatch, n, d, r, nnz, whole):
    """Long segments of sums of mixed vector width take the two-stage sums; gradients against 64 bits on both sides."""
    launches, dg, ref = _backward_with_trace(emu, capfd, monkeypatch, n, d, r, nnz)
    assert any("k_seg_whole" in ln for ln in launches) == whole, launches
    for a, b in zip(dg, ref):  # sums of up to 2049 terms in 32 bits
        assert np.linalg.norm(a - b) <= 2e-6 * np.linalg.norm(b)


@pytest.mark.parametrize("n,d,r,nnz,workgroups", [
    ((2, 20000, 2), (1, 2, 1), (1, 3, 3, 1), 60, 60 + 59),        # 341 slices cleared by a workgroup, then one per prefix
    ((3, 2000, 2), (2, 11, 2), (1, 17, 24, 1), 30, 30 * 10 + 286),  # five column tiles, two of r1; seven slices at a time
    ((2, 16446, 2), (1, 2, 1), (1, 3, 3, 1), 62, 62 + 49), ((2, 16445, 2), (1, 2, 1), (1, 3, 3, 1), 62, 16445),  # the rule's edge
    ((3, 2000, 2), (2, 11, 2), (1, 17, 24, 1), 0, 286),           # no lookup at all
])
def test_core1_gradient_of_mostly_untouched_slices(emu, capfd, monkeypatch, n, d, r, nnz, workgroups):
    """Tables with thousands of i2 that no lookup touched: their slices are cleared by workgroups that take many at a time,
    and only the prefixes' i2 get workgroups of their own; the gradient is written whole and right, also in the
    fused update, which leaves the untouched slices as they are."""
    launches, dg, ref = _backward_with_trace(emu, capfd, monkeypatch, n, d, r, nnz)
    grids = [int(ln.split("grid (")[1].split(",")[0]) for ln in launches if "k_bwd_dg2" in ln]
    assert grids == [workgroups], launches
    for a, b in zip(dg, ref):  # (uninitialised memory went in: every element is written)
        assert np.all(np.isfinite(a)) and np.linalg.norm(a - b) <= 2e-6 * np.linalg.norm(b)
        assert np.array_equal(a == 0, b == 0)


@pytest.mark.parametrize("nnz,grids", [(62, [11808, 4637]), (100, [100 + 49])])
def test_core1_gradient_in_several_launches(capfd, monkeypatch, nnz, grids):
    """More i2 than a launch takes workgroups for, in a build whose launches take 20000: the first launch ends at its limit
    and the second goes on there; with a few lookups more untouched slices the other route takes one."""
    small = _load(emu_build.build_shared(BUILD_DIR, "few_wgs", ["-DTT_MAX_WORKGROUPS=20000"]))
    n = (2, 16445 if nnz == 62 else 16484, 2)
    launches, dg, ref = _backward_with_trace(small, capfd, monkeypatch, n, (1, 2, 1), (1, 3, 3, 1), nnz)
    assert [int(ln.split("grid (")[1].split(",")[0]) for ln in launches if "k_bwd_dg2" in ln] == grids
    for a, b in zip(dg, ref):
        assert np.all(np.isfinite(a)) and np.linalg.norm(a - b) <= 2e-6 * np.linalg.norm(b)
