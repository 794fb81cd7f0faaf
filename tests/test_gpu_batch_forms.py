"""Both forms of a batch in every precision, on either side of the rule that
chooses between them (tests/test_host_routes.py): each request equals the same
request evaluated alone, bit for bit."""
import numpy as np
import pytest

import wlinputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per,side", [(8, 12), (8, 160), (9, 12), (9, 60), (13, 100)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_batch_equals_alone(per, side, prec):
    import paper_1407_7486_amd as wl
    print("[case] batch", per, side, prec, flush=True)
    G = 64
    x, y = wlinputs.polygon_loops(G * per, 24, seed=per)
    rho, T = np.linspace(0.0, 4.0, side), np.geomspace(1e-2, 20.0, side)
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, G)
    try:
        reqs = [dict(kind=k, eB0=2.0, lam=1.2, rho=rho[:n], T=T, spin=s, precision=prec)
                for k, s, n in ((1, 1, side), (2, 0, 3), (0, 1, 2), (3, 1, 1))]
        for q, b in zip(reqs, wl.wl_average_batch(ctx, ens, reqs, full=True)):
            a = wl.wl_average_ex(ctx, ens, wl.field(q["kind"], q["eB0"], q["lam"]), q["rho"],
                                 q["T"], q["spin"], prec)
            for k in wl.RESULT_KEYS:
                assert np.array_equal(a[k], b[k], equal_nan=True), (k, q["kind"])
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)
