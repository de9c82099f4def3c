"""The matrix-core forward on split fp32 numbers (kernels compiled for the CPU, the route taken at every size in a variant of
its own) against 64 bits, and with infinities, NaN and the largest numbers against the arm without a plan."""
import numpy as np
import pytest

import test_cpu_emulation as te
import tt_workloads as wl

pytestmark = te.pytestmark


@pytest.fixture(scope="module")
def emu_split():
    return te._load(te.emu_build.build_shared(te.BUILD_DIR, "split", ["-DTT_DIRECT_MAX_LOOKUPS_32=0", "-DTT_DIRECT_MAX_LOOKUPS_64=0"]))


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
