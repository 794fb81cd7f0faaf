"""Small launches walk each loop with several waves and sum its blocks in the
order of one wave's walk: every output must equal, bit for bit, that of the
same request in a batch, whose kernels give a loop to one wave.  Points per
loop at the edges of the 32-, 8- and single-segment blocks, loops per row that
leave a ragged last row, and grids of one lane, one chunk and a ragged one; a
grid point outside the domain (device grids) must still give NaN."""
import numpy as np
import pytest

import wlinputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wl():
    import paper_1407_7486_amd as wl
    return wl


@pytest.mark.parametrize("n_ppl,per,G,n_rho,n_T", [
    (128, 8, 4, 1, 1),      # shortest that takes it, one grid point
    (135, 11, 8, 5, 13),    # 4 blocks of 32, 7 single segments; ragged chunk
    (255, 1, 3, 8, 8),      # 4 waves, one loop per row
    (257, 25, 16, 8, 8),    # 8 waves, rows of 9, 9 and 7 loops
    (384, 8, 16, 7, 9),     # shortest for every field
    (1003, 3, 5, 3, 50),    # more blocks than waves
    (515, 85, 24, 9, 15),   # 4 waves, rows of 9 loops, the last of 4
    (771, 64, 32, 16, 16),  # 4 waves, even rows (sech^2)
])
def test_walk_equals_one_wave_per_loop(wl, n_ppl, per, G, n_rho, n_T):
    print("[case] walk", n_ppl, per, G, n_rho, n_T, flush=True)
    x, y = wlinputs.polygon_loops(G * per, n_ppl, seed=n_ppl)
    rho, T = np.linspace(0.0, 4.0, n_rho), np.geomspace(1e-2, 20.0, n_T)
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, G)
    try:
        for kind in (0, 1, 2, 3):
            for spin in (0, 1):
                fld = wl.field(kind, 2.0, 1.2)
                one = wl.wl_average_ex(ctx, ens, fld, rho, T, spin, wl.WL_FP32C)
                bat = wl.wl_average_batch(ctx, ens, [dict(
                    kind=kind, eB0=2.0, lam=1.2, rho=rho, T=T, spin=spin,
                    precision=wl.WL_FP32C)], full=True)[0]
                for k in wl.RESULT_KEYS:
                    assert np.array_equal(one[k], bat[k], equal_nan=True), (k, kind, spin)
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)


def test_walk_domain(wl):
    import torch
    print("[case] walk domain", flush=True)
    x, y = wlinputs.polygon_loops(64, 400, seed=4)
    ctx = wl.wl_create(0, None)
    ens = wl.wl_ensemble_upload(ctx, x, y, 8)
    try:
        rho = torch.tensor([0.5, -1.0, 1.0], dtype=torch.float64, device="cuda")
        T = torch.tensor([0.3, float("nan"), 2.0], dtype=torch.float64, device="cuda")
        sums = torch.empty(8, 3, 3, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        wl.wl_average_async(ctx, ens, wl.field(1, 2.0, 1.2), rho, T, 1, wl.WL_FP32C, None,
                            None, sums)
        torch.cuda.synchronize()
        got = sums.cpu().numpy()
        want = wl.wl_average(ctx, ens, wl.field(1, 2.0, 1.2), np.array([0.5, 1.0]),
                             np.array([0.3, 2.0]), 1, wl.WL_FP32C)[2]
        assert np.array_equal(got[:, ::2, ::2], want)
        assert np.isnan(got[:, 1, :]).all() and np.isnan(got[:, :, 1]).all()
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)
