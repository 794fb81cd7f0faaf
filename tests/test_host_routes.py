"""Which kernels the host code chooses, on the CPU (fake_hip): the two forms of
a batch at the sizes where one side was measured to be the faster, and the
walk of small launches for the shapes of test_gpu_walk.py."""
import pytest

import fake_hip

BATCH = [
    # loops per group, groups, grid side, requests, precision, wide
    # FP64 and rows that leave waves idle: narrow beyond a fraction of a round
    (85, 24, 16, 13, 2, 0), (85, 24, 16, 16, 2, 0), (85, 24, 16, 4, 2, 0),
    (85, 24, 16, 21, 1, 0), (85, 24, 16, 21, 0, 0), (6, 340, 16, 6, 0, 0),
    (64, 64, 16, 2, 2, 0), (42, 48, 16, 9, 1, 0),
    (85, 24, 8, 1, 0, 1), (64, 64, 8, 1, 2, 1), (85, 24, 8, 1, 2, 1),
    # rows that keep them busy: wide up to some rounds
    (64, 64, 16, 1, 0, 1), (64, 64, 16, 4, 1, 1), (64, 64, 16, 16, 0, 1),
    (64, 64, 16, 40, 0, 0), (64, 64, 16, 40, 1, 0),
    (13, 128, 16, 8, 0, 1), (4, 512, 16, 8, 0, 1), (1, 2048, 16, 4, 0, 1),
    # tests/test_gpu_split.py
    (8, 64, 160, 1, 2, 0), (9, 64, 160, 1, 0, 0),
]


def test_batch_forms():
    out = fake_hip.run("""
ctx = wl.wl_create(0, 0x1000)
for per, G, side, n, prec, want in %r:
    ens = wl.wl_ensemble_upload(ctx, np.ones((per * G, 16), np.float32),
                                np.ones((per * G, 16), np.float32), G)
    reqs = [dict(kind=1, eB0=1.0, lam=1.0, rho=np.linspace(0, 4, side),
                 T=np.geomspace(1e-2, 10, side), spin=1, precision=prec)] * n
    clear()
    wl.wl_average_batch(ctx, ens, reqs)
    head = [c.split() for c in calls() if c.startswith("h2d")][0]
    assert int(head[3]) == n  # the header: requests, wide
    if int(head[4]) != want:
        print(per, G, side, n, prec, "wide", head[4])
    wl.wl_ensemble_free(ens)
wl.wl_destroy(ctx)
""" % BATCH)
    assert out == "", out


WALK = [
    # n_ppl, loops per group, groups, n_rho, n_T, kinds that take k_walk
    (128, 8, 4, 1, 1, (1, 2)), (135, 11, 8, 5, 13, (1, 2)), (255, 1, 3, 8, 8, (1, 2)),
    (257, 25, 16, 8, 8, (1, 2)), (384, 8, 16, 7, 9, (0, 1, 2, 3)),
    (1003, 3, 5, 3, 50, (0, 1, 2, 3)), (515, 85, 24, 9, 15, (1, 2)),
    (771, 64, 32, 16, 16, (1,)),
    (127, 8, 4, 1, 1, ()), (383, 8, 16, 7, 9, (1, 2)),
]


@pytest.mark.parametrize("n_ppl,per,G,n_rho,n_T,kinds", WALK)
def test_walk_of_small_launches(n_ppl, per, G, n_rho, n_T, kinds):
    fake_hip.run("""
n_ppl, per, G, n_rho, n_T, kinds = %r
ctx = wl.wl_create(0, 0x1000)
ens = wl.wl_ensemble_upload(ctx, np.ones((per * G, n_ppl), np.float32),
                            np.ones((per * G, n_ppl), np.float32), G)
for kind in range(4):
    clear()
    wl.wl_average(ctx, ens, wl.field(kind, 2.0, 1.2), np.linspace(0, 4, n_rho),
                  np.geomspace(1e-2, 20, n_T), 1, wl.WL_FP32C)
    walk = any("k_walkI" in c for c in calls())
    assert walk == (kind in kinds) and walk != any("k_average" in c for c in calls()), kind
""" % ((n_ppl, per, G, n_rho, n_T, kinds),))


SPLIT = [
    # n_ppl, loops per group, groups, n_rho, n_T, then the waves of a workgroup in
    # FP64: k_average and k_disc in the constant field, the same in sech^2
    (2048, 64, 64, 32, 32, 8, 8, 8, 8),      # long walks
    (1000, 85, 24, 40, 33, 4, 4, 8, 8),      # rows of 9
    (1000, 5, 24, 8, 8, 5, 5, 5, 5), (1000, 1, 24, 8, 8, 1, 1, 1, 1),
    (256, 128, 64, 40, 33, 4, 4, 8, 8),      # 21504 items
    (128, 256, 64, 40, 33, 1, 1, 8, 8), (64, 512, 64, 40, 33, 1, 1, 4, 4),
    (16, 1024, 64, 40, 33, 1, 1, 1, 1), (16, 64, 64, 16, 16, 4, 4, 8, 8),  # 2048 items
    (12, 2496, 8, 9, 9, 8, 8, 8, 8), (8, 1, 64, 16, 16, 1, 1, 1, 1),
]


@pytest.mark.parametrize("n_ppl,per,G,n_rho,n_T,ca,cd,sa,sd", SPLIT)
def test_waves_of_an_item(n_ppl, per, G, n_rho, n_T, ca, cd, sa, sd):
    fake_hip.run("""
n_ppl, per, G, n_rho, n_T, ca, cd, sa, sd = %r
ctx = wl.wl_create(0, 0x1000)
ens = wl.wl_ensemble_upload(ctx, np.ones((per * G, n_ppl), np.float32),
                            np.ones((per * G, n_ppl), np.float32), G)
rho, T = np.linspace(0, 4, n_rho), np.geomspace(1e-2, 20, n_T)
def waves(name):
    return [int(c.split("x")[-1]) // 64 for c in calls() if name in c][0]
for kind, want, disc in ((0, ca, cd), (1, sa, sd)):
    clear()
    wl.wl_average(ctx, ens, wl.field(kind, 2.0, 1.2), rho, T, 1, wl.WL_FP64)
    assert waves("k_average") == want, (kind, waves("k_average"))
    if n_ppl %% 4 == 0:
        clear()
        wl.wl_discretisation(ctx, ens, wl.field(kind, 2.0, 1.2), rho, T, 1, wl.WL_FP64)
        assert waves("k_disc") == disc, (kind, waves("k_disc"))
""" % ((n_ppl, per, G, n_rho, n_T, ca, cd, sa, sd),))
