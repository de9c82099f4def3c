"""The matrix-core forward on split fp32 numbers (kernels compiled for the CPU, the route taken at every size in a variant of
its own) against 64 bits, and with infinities, NaN and the largest numbers against the arm without a plan."""
import ctypes

import numpy as np
import pytest

import test_cpu_emulation as te
import tt_workloads as wl

pytestmark = te.pytestmark


@pytest.fixture(scope="module")
def emu_split():
    return te._load(te.emu_build.build_shared(te.BUILD_DIR, "split", ["-D%s_%d=0" % (m, r) for r in (32, 64)
                                                                for m in ("TT_DIRECT_MAX_LOOKUPS", "TT_FORWARD_SPLIT_ABOVE")]))


@pytest.fixture(scope="module")
def emu():
    return te._load(te.emu_build.build_shared(te.BUILD_DIR))  # short batches: the fp32 instruction


def _problem(r, n, nb, seed):
    shape, cores, idx, off, grad = wl.small_random_problem(seed, n=n, d=(4, 8, 4), r=(1, r, r, 1), num_bags=nb, max_len=3, sigma=0.2)
    return shape, [np.array(c) for c in cores], idx, off, grad


def _exact(shape, cores, idx, off):
    n, d, r = shape.n, shape.d, shape.r
    c = [x.astype(np.float64).reshape(r[k], n[k], d[k], r[k + 1]) for k, x in enumerate(cores)]
    out = np.zeros((len(off) - 1, shape.dim))
    for b in range(len(off) - 1):
        for row in idx[off[b]:off[b + 1]]:
            i1, i2, i3 = row // (n[1] * n[2]), row // n[2] % n[1], row % n[2]
            p = np.tensordot(np.tensordot(c[0][0, i1], c[1][:, i2], 1), c[2][:, i3], 1)
            out[b] += p.reshape(-1)
    return out


# prefixes per i2: one, four, five, eight, nine and more (half tiles, whole chunks, a second chunk)
@pytest.mark.parametrize("r", [32, 64])
@pytest.mark.parametrize("n,nb", [((1, 3, 2), 20), ((4, 2, 3), 60), ((5, 1, 3), 60), ((8, 1, 2), 80), ((9, 2, 2), 120)])
def test_error_against_64_bits(emu_split, r, n, nb):
    shape, cores, idx, off, grad = _problem(r, n, nb, 11 * r + n[0])
    rng = np.random.default_rng(r)
    cores = [(c * 10.0 ** rng.uniform(-3, 3, c.shape)).astype(np.float32) for c in cores]
    out = te._run(emu_split, shape, cores, idx, off, grad, 0.0)["plan"][0]
    # every path is a product of three numbers (two roundings, 2^-24 for the terms the split leaves out) in two sums of r
    # terms and one of at most three rows: below (2 + 1 + 2 * r + 3) * 2^-24 of the sum of absolute paths, twice over
    bound = 2 * (2 * r + 6) * 2.0 ** -24 * _exact(shape, [np.abs(c) for c in cores], idx, off)
    assert (np.abs(out - _exact(shape, cores, idx, off)) <= bound).all()


@pytest.mark.parametrize("r", [32, 64])
@pytest.mark.parametrize("core", [0, 1, 2])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_infinities_nan_and_the_largest_numbers(emu_split, r, core, value):
    shape, cores, idx, off, grad = _problem(r, (9, 2, 3), 60, 5)
    cores[core].reshape(-1)[[3, cores[core].size // 2]] = value
    with np.errstate(all="ignore"):
        res = te._run(emu_split, shape, cores, idx, off, grad, 0.0)
    got, want = res["plan"][0], res["naive"][0]
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    fin = np.isfinite(want)
    if value == value and abs(value) < np.inf:
        assert fin.any()
    assert np.allclose(got[fin], want[fin], rtol=1e-4, atol=1e-5 * np.abs(want[fin]).max(initial=0.0))


def _products(r, n, seed, terms):
    """A problem whose bag sums are the prefix products (core 2 picks one r2 per column), `terms` non-zero r1 a row of core 0;
    every row once, and the products in 64 bits."""
    rng = np.random.default_rng(seed)
    n = (n[0], n[1], r // 4)
    shape = wl.TableShape(n[0] * n[1] * n[2], n, (4, 8, 4), (1, r, r, 1))
    c0 = rng.standard_normal((n[0], 4, r)) * (rng.random((n[0], 4, r)).argsort(-1) < terms)
    c1 = rng.standard_normal((r, n[1], 8, r))
    cores = [c0.astype(np.float32), c1.astype(np.float32), np.eye(r, dtype=np.float32).reshape(r, n[2], 4)]
    idx = np.arange(shape.num_rows)
    return shape, cores, idx, np.arange(shape.num_rows + 1)


def _product_sums(emu, problem):
    (lib, binding), (shape, raw, idx, off) = emu, problem
    cores = [te._aligned(4 * c.size).view(np.float32) for c in raw]
    for c, x in zip(cores, raw):
        c[:] = x.reshape(-1)
    table, nnz, plan = te._table(binding, shape, cores), len(idx), binding.CPlan()
    ws = te._aligned(lib.tt_workspace_bytes(ctypes.byref(table), nnz, nnz))
    assert lib.tt_index_reorder(ctypes.byref(table), te._ptr(idx), te._ptr(off), nnz, nnz, None, te._ptr(ws), ws.nbytes,
                                ctypes.byref(plan), None) == 0
    out = np.full((nnz, shape.dim), np.nan, np.float32)
    assert lib.tt_emb_bag_forward(ctypes.byref(table), ctypes.byref(plan), te._ptr(idx), te._ptr(off), nnz, nnz, te._ptr(out), None) == 0
    return out


def _exact_products(problem):
    shape, (c0, c1, _), idx, _ = problem
    p = np.tensordot(c0.astype(np.float64), c1.astype(np.float64), 1).transpose(0, 2, 1, 3, 4)  # [i1][i2][j1][j2][r2]
    p = p.reshape(-1, 32, shape.n[2], 4).transpose(0, 2, 1, 3)
    return p.reshape(len(idx), 128)


# One term: a product rounded once by either, so the errors are the same to half a percent (each of the eight terms left out shows).
# More terms: fewer roundings at full size.  (Emulated, the instruction adds its terms one after the other in fp32; the GPU
# test has the hardware's sums.)
@pytest.mark.parametrize("r", [32, 64])
@pytest.mark.parametrize("terms,most", [(1, 1.005), (2, 1.005), (4, 1.005), (64, 1.05)])
def test_no_less_exact_than_the_fp32_instruction(emu, emu_split, r, terms, most):
    problem = _products(r, (9, 2), 3 * r + terms, terms)
    want = _exact_products(problem)
    whole, split = (np.linalg.norm(_product_sums(e, problem) - want) / np.linalg.norm(want) for e in (emu, emu_split))
    assert split <= most * whole and split <= 6e-7


# core 0 so small, and core 1 so large, that parts or products of parts would be denormal: the fp32 instruction's bits, also from
# the second chunk of prefixes on only, and from a strip on
@pytest.mark.parametrize("r", [32, 64])
@pytest.mark.parametrize("where", ["all", "chunk", "strip"])
def test_operands_too_small_to_split(emu, emu_split, r, where):
    problem = _products(r, (19, 2), r, r)
    c0, c1, _ = problem[1]
    if where == "all":
        c0 *= np.float32(2.0 ** -116)
        c1 *= np.float32(2.0 ** 100)
    elif where == "chunk":
        c0[8:, 2, 5] *= np.float32(2.0 ** -100)
    else:
        c1[3, :, 7, 1] *= np.float32(2.0 ** -100)  # (the last strip; the others are split)
    whole, split = (_product_sums(e, problem).reshape(19, -1, 4, 8, 4) for e in (emu, emu_split))
    same = slice(8, None) if where == "chunk" else slice(None)
    cols = slice(8 - 256 // r, 8) if where == "strip" else slice(None)
    assert np.array_equal(whole[same, :, :, cols], split[same, :, :, cols])
    want = _exact_products(problem).reshape(whole.shape)
    assert np.abs(split - want).max() <= 1e-6 * np.abs(want).max()
