"""Buffers that the library makes on first use do not end the capture of another
stream (fake_hip: an allocation then ends it unless the thread relaxed its mode),
and a call without room for them still runs."""
import fake_hip

SETUP = """
ctx = wl.wl_create(0, 0x1000)
x = np.ones((256, 512), np.float32)
ens = wl.wl_ensemble_upload(ctx, x, x, 8)
fld = wl.field(1, 1.0, 1.0)
rho, T = np.linspace(0, 4, 3), np.geomspace(1e-2, 10, 7)
wl.wl_average(ctx, ens, fld, rho, T, 1, wl.WL_FP64)  # everything but the walk's room
"""


def test_another_streams_capture_goes_on():
    fake_hip.run(SETUP + """
fake.fake_foreign_capture(1)
clear()
wl.wl_average(ctx, ens, fld, rho, T, 1, wl.WL_FP32C)
assert any("k_walk" in c for c in calls())
assert fake.fake_foreign_capture_left()
""")


def test_without_room_each_loop_is_walked_by_one_wave():
    fake_hip.run(SETUP + """
fake.fake_limit(fake.fake_used())
clear()
wl.wl_average(ctx, ens, fld, rho, T, 1, wl.WL_FP32C)
assert any("k_average" in c for c in calls())
fake.fake_limit(1 << 38)
clear()
wl.wl_average(ctx, ens, fld, rho, T, 1, wl.WL_FP32C)
assert any("k_walk" in c for c in calls())
""")
