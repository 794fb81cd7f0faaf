"""Host arrays travel through 8 MiB halves of a pinned staging buffer, and
freed ensembles' memory serves the next ones: results whose arrays end below,
at and beyond a half's edge, and ensembles of changing shapes in reused
memory, against the same values computed in small pieces or by numpy."""
import sys

import numpy as np
import pytest

import wlinputs

pytestmark = pytest.mark.gpu

HALF = (8 << 20) // 8  # doubles in a half


@pytest.fixture(scope="module")
def wl():
    import paper_1407_7486_amd as wl
    return wl


@pytest.fixture(scope="module")
def ctx(wl):
    c = wl.wl_create(0, None)
    yield c
    wl.wl_destroy(c)


@pytest.mark.parametrize("n_pts", [1, 4095, 4096, 4097])
def test_per_loop_across_halves(wl, ctx, n_pts):
    print("[case] staging", n_pts, flush=True)
    sys.stdout.flush()
    nl = HALF // 4096  # 256 loops: 4096 points fill a half per array
    x, y = wlinputs.polygon_loops(nl, 16, seed=2)
    ens = wl.wl_ensemble_upload(ctx, x, y, 1)
    try:
        fld = wl.field(2, 1.5, 0.8)
        rho, T = np.linspace(0.0, 2.0, n_pts), np.array([0.7])
        got = wl.wl_per_loop(ctx, ens, fld, rho, T, 1, wl.WL_FP64, 0, nl)
        for a in range(0, nl, 64):
            part = wl.wl_per_loop(ctx, ens, fld, rho, T, 1, wl.WL_FP64, a, 64)
            for u, v in zip(got, part):
                assert np.array_equal(u[a:a + 64], v)
    finally:
        wl.wl_ensemble_free(ens)


@pytest.mark.parametrize("n_units", [1000, HALF // 8, 3 * HALF // 8 + 24])
def test_regroup_across_halves(wl, ctx, n_units):
    print("[case] staged regroup", n_units, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(n_units)
    X = rng.integers(-1000, 1000, (n_units, 8)).astype(np.float64)  # exact sums
    perms = np.stack([rng.permutation(n_units) for _ in range(3)])
    which = np.array([0, 1, 2, 0, 1, 2, 1, 1], dtype=np.int32)
    got = wl.wl_regroup(ctx, X, perms, 8, which)
    want = np.stack([X[perms[w], p].reshape(8, -1).sum(1) for p, w in enumerate(which)], axis=1)
    assert np.array_equal(got, want)


def test_ensembles_in_reused_memory(wl, ctx):
    print("[case] reused ensemble memory", flush=True)
    sys.stdout.flush()
    rho, T = np.linspace(0.0, 2.0, 3), np.geomspace(0.1, 5.0, 5)
    fld = wl.field(1, 1.0, 1.0)
    for nl, n in ((64, 256), (64, 250), (48, 300), (64, 64), (64, 256)):
        x, y = wlinputs.polygon_loops(nl, n, seed=nl + n)
        ens = wl.wl_ensemble_upload(ctx, x, y, 8)
        try:
            dx, dy = wl.wl_ensemble_download(ens, 0, nl)
            assert np.array_equal(dx, x) and np.array_equal(dy, y)
            mean = wl.wl_average(ctx, ens, fld, rho, T, 1, wl.WL_FP64)[0]
        finally:
            wl.wl_ensemble_free(ens)
        fresh = wl.wl_create(0, None)  # nothing kept
        ens = wl.wl_ensemble_upload(fresh, x, y, 8)
        try:
            assert np.array_equal(mean, wl.wl_average(fresh, ens, fld, rho, T, 1, wl.WL_FP64)[0])
        finally:
            wl.wl_ensemble_free(ens)
            wl.wl_destroy(fresh)
