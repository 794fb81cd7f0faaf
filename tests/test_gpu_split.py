"""The loops of an item are dealt to up to 8 waves: the results do not depend
on which loops share a row's workgroup rounds.  An ensemble evaluated with
its rows' loops in one order of rounds (any grid) must equal, bit for bit,
the sums of its loops' own values (one loop per group: one wave per item)
added in loop order, for loop counts per row below, at and between the
multiples of 8, and the ragged last chunk of a grid must equal the same
points of a larger one."""
import sys

import numpy as np
import pytest

import wlinputs

pytestmark = pytest.mark.gpu

RHO = np.linspace(0.0, 4.0, 128)
T = np.geomspace(1e-2, 20.0, 64)
T_RAGGED = T[::5]
J, K = np.array([0, 3, 50, 90, 127]), np.arange(0, 64, 5)  # 5 x 13 = 65 points


@pytest.fixture(scope="module")
def wl():
    import paper_1407_7486_amd as wl
    return wl


@pytest.mark.parametrize("per", [1, 3, 8, 11])
@pytest.mark.parametrize("n_ppl", [24, 100])
def test_sums_do_not_depend_on_the_split(wl, per, n_ppl):
    print("[case] split", per, "loops per row,", n_ppl, "points", flush=True)
    sys.stdout.flush()
    G = 64
    x, y = wlinputs.polygon_loops(G * per, n_ppl, seed=11)
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, G)
    try:
        for kind, spin in ((1, 1), (2, 0), (0, 1), (3, 1)):
            fld = wl.field(kind, 2.0, 1.2)
            for prec in (wl.WL_FP32, wl.WL_FP64, wl.WL_FP32K):
                # rows of `per` loops (fewer than 16: one row per group)
                # against the loops' values added in order
                got = wl.wl_average(ctx, ens, fld, RHO[J], T[K], spin, prec)[2]
                wl.wl_ensemble_set_groups(ens, G * per)
                one = wl.wl_average(ctx, ens, fld, RHO[J], T[K], spin, prec)[2]
                wl.wl_ensemble_set_groups(ens, G)
                want = np.zeros_like(got)
                for k in range(per):
                    want += one[k::per]
                assert np.array_equal(got, want), (kind, spin, prec)
            for prec in (wl.WL_FP32C, wl.WL_FP32, wl.WL_FP64, wl.WL_FP32K):
                a = wl.wl_average_ex(ctx, ens, fld, RHO, T, spin, prec)
                b = wl.wl_average_ex(ctx, ens, fld, RHO[J], T[K], spin, prec)
                for k in ("group_sums", "scale", "fp_err", "escalated", "mean", "err"):
                    u = a[k][..., J[:, None], K]
                    assert np.array_equal(u, b[k], equal_nan=True), (k, kind, spin, prec)
            for mode in (wl.WL_DISC_PAPER, wl.WL_DISC_FULL):
                for prec in (wl.WL_FP32C, wl.WL_FP64):
                    a = wl.wl_discretisation(ctx, ens, fld, RHO, T, spin, prec, mode)
                    b = wl.wl_discretisation(ctx, ens, fld, RHO[J], T[K], spin, prec, mode)
                    for u, v in zip(a, b):
                        assert np.array_equal(u[..., J[:, None], K], v, equal_nan=True)
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)


@pytest.mark.parametrize("per,prec,big", [(1, 0, False), (3, 0, False), (5, 2, False),
                                          (11, 1, False), (8, 2, True), (9, 0, True)])
def test_batch_forms_equal_alone(wl, per, prec, big):
    """A small batch deals an item's loops to a team of waves (1, 2, 4 or 8,
    by the loops per row), a large one gives each wave an item: both equal
    the request evaluated alone, bit for bit."""
    print("[case] batch forms", per, prec, big, flush=True)
    sys.stdout.flush()
    G = 64
    x, y = wlinputs.polygon_loops(G * per, 24, seed=3)
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, G)
    try:
        rho = np.linspace(0.0, 4.0, 160) if big else RHO[J]
        T = np.geomspace(1e-2, 20.0, 160) if big else T_RAGGED
        reqs = [dict(kind=1, eB0=2.0, lam=1.2, rho=rho, T=T, spin=1, precision=prec),
                dict(kind=2, eB0=1.0, lam=0.7, rho=RHO[:3], T=T_RAGGED, spin=0,
                     precision=prec)]
        for q, b in zip(reqs, wl.wl_average_batch(ctx, ens, reqs, full=True)):
            a = wl.wl_average_ex(ctx, ens, wl.field(q["kind"], q["eB0"], q["lam"]), q["rho"],
                                 q["T"], q["spin"], prec)
            for k in wl.RESULT_KEYS:
                assert np.array_equal(a[k], b[k], equal_nan=True), k
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)
