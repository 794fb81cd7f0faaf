"""The FP64 recomputation of a batch takes the flagged points of every field
and spin in one kernel: a batch with requests of all of them, flagged or not,
in two orders, must equal each request evaluated alone, bit for bit."""
import numpy as np
import pytest

import wlinputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ppl,order", [(512, 1), (1001, -1)])
def test_every_variant_in_one_batch(n_ppl, order):
    import paper_1407_7486_amd as wl
    print("[case] recompute", n_ppl, order, flush=True)
    x, y = wlinputs.polygon_loops(512, n_ppl, seed=21)
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, 16)
    try:
        reqs = [dict(kind=kind, eB0=eB0, lam=4.0, rho=np.linspace(0.0, 8.0, 5 + kind),
                     T=np.geomspace(1e-2, 10.0, 9 + spin), spin=spin, precision=wl.WL_FP32C)
                for kind in (0, 1, 2, 3) for spin in (0, 1) for eB0 in (0.1, 20.0)][::order]
        flagged = set()
        for q, b in zip(reqs, wl.wl_average_batch(ctx, ens, reqs, full=True)):
            a = wl.wl_average_ex(ctx, ens, wl.field(q["kind"], q["eB0"], q["lam"]), q["rho"],
                                 q["T"], q["spin"], wl.WL_FP32C)
            for k in wl.RESULT_KEYS:
                assert np.array_equal(a[k], b[k], equal_nan=True), (k, q["kind"], q["spin"])
            if b["escalated"].any():
                flagged.add((q["kind"], q["spin"]))
        assert len(flagged) > 1  # several variants share the kernel
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)
