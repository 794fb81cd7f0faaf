"""The FP64 walk's geometry stays unscaled.

Precision: the spin exponents of the Gaussian tube against long double.  The
kernel's steps carried out in numpy on these inputs are 0.93e-15 and 0.96e-15 off
(relative rms over loops and grid points); with rho_cm and sqrt(T) scaled to
exp2's units beforehand 2.0e-15 and 2.1e-15, since a lane's segments then share
the rounding of the scaled values.  The bound lies between, 1.25e-15.

Range: a tube far narrower than 1e-154 carries no flux, so every loop gives 1
(the scaled radius overflowed to NaN there)."""
import numpy as np
import pytest

import wlinputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wl():
    import paper_1407_7486_amd as wl
    return wl


@pytest.mark.parametrize("seed", [1, 2])
def test_spin_exponents_against_long_double(wl, seed):
    print("[case] fp64 spin exponents", seed, flush=True)
    LD = np.longdouble
    n, lam, eB0 = 1024, 1.5, 1.0
    rng = np.random.default_rng(seed)
    z = rng.normal(size=(2, 48, n)).cumsum(2) * np.sqrt(2.0 / n)
    z -= z[:, :, -1:] * (np.arange(1, n + 1) / n)
    z -= z.mean(2, keepdims=True)
    x, y = z.astype(np.float32)
    rho = rng.uniform(0.0, 5.0 * lam, 40)
    T = np.exp(rng.uniform(np.log(0.1), np.log(50.0), 40))
    X, Y = x.astype(LD), y.astype(LD)
    mx, my = (X + np.roll(X, -1, 1)) / 2, (Y + np.roll(Y, -1, 1)) / 2
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, 1)
    try:
        sq = 0.0
        for r, t in zip(rho, T):
            got = wl.wl_per_loop(ctx, ens, wl.field(wl.WL_GAUSS, eB0, lam), np.array([r]),
                                 np.array([t]), 1, wl.WL_FP64, 0, 48)[1][:, 0, 0]
            r, t = LD(r), LD(t)
            v = ((r + np.sqrt(t) * mx) ** 2 + t * my ** 2) / LD(lam) ** 2
            want = t / n * (LD(eB0) * np.exp(-v)).sum(1)
            sq += float((((got - want) / want) ** 2).mean()) / 40
        print("relative rms %.3e" % np.sqrt(sq), flush=True)
        assert np.sqrt(sq) < 1.25e-15
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)


@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("spin", [0, 1])
def test_tube_without_flux(wl, kind, spin):
    print("[case] fp64 narrow tube", kind, spin, flush=True)
    x, y = wlinputs.polygon_loops(32, 100, seed=3)
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, 4)
    try:
        rho, T = np.array([0.3, 2.0]), np.array([0.5, 10.0])
        fld = wl.field(kind, 1.0, 1e-158)
        mean, err, _ = wl.wl_average(ctx, ens, fld, rho, T, spin, wl.WL_FP64)
        assert np.abs(mean - 1.0).max() < 1e-12 and np.abs(err).max() < 1e-12
        ph, _, w = wl.wl_per_loop(ctx, ens, fld, rho, T, spin, wl.WL_FP64, 0, 32)
        assert np.abs(ph).max() < 1e-12 and np.abs(w - 1.0).max() < 1e-12
        lv = wl.wl_discretisation(ctx, ens, fld, rho, T, spin, wl.WL_FP64)[0]
        assert np.abs(lv - 1.0).max() < 1e-12
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)
