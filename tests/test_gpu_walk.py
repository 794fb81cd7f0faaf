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


@pytest.mark.parametrize("warm_fp64", [False, True])
def test_walk_captured(wl, warm_fp64):
    """A captured small launch, replayed between eager launches of other sizes,
    keeps giving the eager result: the loops' terms have a fixed place.  Warmed
    up in FP64 only, that place does not exist yet and may not be allocated
    under capture: the captured launch walks each loop with one wave."""
    import torch
    print("[case] walk captured", warm_fp64, flush=True)
    x, y = wlinputs.polygon_loops(256, 600, seed=6)
    st = torch.cuda.Stream()
    ctx = wl.wl_create(0, st.cuda_stream)
    ens = wl.wl_ensemble_upload(ctx, x, y, 8)
    fld = wl.field(1, 2.0, 1.2)

    def dev(*shape):
        return torch.zeros(*shape, dtype=torch.float64, device="cuda")

    def grid(n_rho, n_T):
        return (torch.linspace(0.0, 4.0, n_rho, dtype=torch.float64, device="cuda"),
                torch.logspace(-2.0, 1.0, n_T, dtype=torch.float64, device="cuda"),
                dev(8, n_rho, n_T), dev(n_rho, n_T), dev(n_rho, n_T))

    def run(g, prec):
        rho, T, sums, mean, err = g
        wl.wl_average_async(ctx, ens, fld, rho, T, 1, prec, mean, err, sums)

    try:
        small, other = grid(4, 16), grid(8, 24)
        want = wl.wl_average(ctx, ens, fld, small[0].cpu().numpy(), small[1].cpu().numpy(), 1,
                             wl.WL_FP32C) if not warm_fp64 else None
        torch.cuda.synchronize()
        run(small, wl.WL_FP64 if warm_fp64 else wl.WL_FP32C)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            run(small, wl.WL_FP32C)
        for k in range(3):
            if not warm_fp64:  # (a larger scratch would move the captured one)
                run(grid(2, 16), wl.WL_FP32C)
            for a in small[2:]:
                a.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = [a.cpu().numpy() for a in (small[3], small[4], small[2])]
            if want is None:
                want = got
            for u, v in zip(got, want):
                assert np.array_equal(u, v), k
        del graph
        run(other, wl.WL_FP32C)
        eager = wl.wl_average(ctx, ens, fld, small[0].cpu().numpy(), small[1].cpu().numpy(), 1,
                              wl.WL_FP32C)
        for u, v in zip(want, eager):
            assert np.array_equal(u, v)
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)
