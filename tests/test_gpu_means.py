"""Column means and the sample split of wl_correlation at the edges of their
launch rules, against the oracle.

Means are taken in blocks of 16 columns by 64 row slots; rows are split into
blocks from 2049 rows on, and for one or few output tiles the Gram sums are
split in up to 64 sample ranges.  Both sides are FP64 and differ in the order
of the sums only: 1e-11 absolute, as for the other shapes.  A column that is
constant has no deviation, whatever its value and however its rows are split:
its coefficients are 0/0."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wl():
    import paper_1407_7486_amd as wl
    return wl


@pytest.fixture(scope="module")
def ctx(wl):
    c = wl.wl_create(0, None)
    yield c
    wl.wl_destroy(c)


@pytest.mark.parametrize("n_units,n_pts", [
    (63, 16), (64, 17), (65, 15),     # one row slot short, full, over
    (2048, 33), (2049, 31),           # one block of rows, two
    (4097, 1), (9001, 130),           # one column; three tiles, many ranges
])
def test_means_and_ranges(wl, ctx, n_units, n_pts):
    print("[case] means", n_units, n_pts, flush=True)
    rng = np.random.default_rng(n_units * 1000 + n_pts)
    X = rng.standard_normal((n_units, n_pts)) + 0.5 * rng.standard_normal((n_units, 1))
    X = X * rng.uniform(0.1, 10, n_pts) + rng.uniform(-5, 5, n_pts)
    got = wl.wl_correlation(ctx, X)
    np.testing.assert_allclose(got, oracle.correlation(X), rtol=0, atol=1e-11)
    assert np.array_equal(got, got.T)


@pytest.mark.parametrize("n_units", [65, 2049])
def test_constant_column(wl, ctx, n_units):
    print("[case] constant column", n_units, flush=True)
    X = np.random.default_rng(n_units).standard_normal((n_units, 18))
    X[:, 17] = 0.1
    got = wl.wl_correlation(ctx, X)
    assert np.isnan(got[17]).all() and np.isnan(got[:, 17]).all()
    np.testing.assert_allclose(got[:17, :17], oracle.correlation(X[:, :17]), rtol=0, atol=1e-11)
