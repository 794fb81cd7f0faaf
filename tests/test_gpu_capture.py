"""A small evaluation on the context's stream while torch captures another one:
the capture holds (the room for the loops' terms is made by this call), and the
evaluation gives what it gives elsewhere."""
import numpy as np
import pytest

import wlinputs

pytestmark = pytest.mark.gpu


def test_evaluation_beside_a_capture():
    import torch

    import paper_1407_7486_amd as wl
    print("[case] evaluation beside a capture", flush=True)
    x, y = wlinputs.polygon_loops(256, 600, seed=6)
    st = torch.cuda.Stream()
    ctx = wl.wl_create(0, st.cuda_stream)
    ens = wl.wl_ensemble_upload(ctx, x, y, 8)
    fld = wl.field(1, 2.0, 1.2)
    try:
        rho = torch.linspace(0.0, 4.0, 4, dtype=torch.float64, device="cuda")
        T = torch.logspace(-2.0, 1.0, 16, dtype=torch.float64, device="cuda")
        mean, err = (torch.zeros(4, 16, dtype=torch.float64, device="cuda") for _ in range(2))
        sums = torch.zeros(8, 4, 16, dtype=torch.float64, device="cuda")
        a = torch.zeros(8, device="cuda")
        torch.cuda.synchronize()
        # makes the scratch, which a plain FP32 call shares
        wl.wl_average_async(ctx, ens, fld, rho, T, 1, wl.WL_FP32, mean, err, sums)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            a += 1.0
            wl.wl_average_async(ctx, ens, fld, rho, T, 1, wl.WL_FP32C, mean, err, sums)
            a += 1.0
        torch.cuda.synchronize()
        for k in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert float(a.min()) == float(a.max()) == 2.0 * (k + 1)
        want = wl.wl_average(ctx, ens, fld, rho.cpu().numpy(), T.cpu().numpy(), 1, wl.WL_FP32C)
        for u, v in zip((mean, err, sums), want):
            assert np.array_equal(u.cpu().numpy(), v)
        del graph
    finally:
        wl.wl_ensemble_free(ens)
        wl.wl_destroy(ctx)
