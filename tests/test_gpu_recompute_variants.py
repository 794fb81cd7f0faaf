"""A batch's FP64 recomputation takes every field and spin in one kernel: here
each of the eight variants has flagged points, and its recomputed means agree
with an evaluation in FP64 within the mean bar of wl_tol.py."""
import numpy as np
import pytest

import wlinputs
from wl_tol import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ppl", [512, 1001])
def test_flagged_points_of_every_variant(n_ppl):
    import paper_1407_7486_amd as wl
    print("[case] recompute variants", n_ppl, flush=True)
    x, y = wlinputs.polygon_loops(512, n_ppl, seed=21)
    rho, T = np.linspace(0.0, 8.0, 5), np.geomspace(1e-2, 10.0, 9)
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, 16)
    try:
        reqs = [dict(kind=kind, eB0=20.0, lam=4.0, rho=rho, T=T, spin=spin,
                     precision=wl.WL_FP32C) for kind in (2, 0, 3, 1) for spin in (1, 0)]
        flagged = set()
        for q, b in zip(reqs, wl.wl_average_batch(ctx, ens, reqs, full=True)):
            ref = wl.wl_average_ex(ctx, ens, wl.field(q["kind"], 20.0, 4.0), rho, T, q["spin"],
                                   wl.WL_FP64)
            at = b["escalated"] > 0
            if at.any():
                flagged.add((q["kind"], q["spin"]))
            dev = np.abs(b["mean"] - ref["mean"]) / ref["scale"]
            assert dev[at].max(initial=0.0) <= TOL[wl.WL_FP32C]["mean"], (q["kind"], q["spin"])
        assert flagged == {(k, s) for k in range(4) for s in (0, 1)}
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)
