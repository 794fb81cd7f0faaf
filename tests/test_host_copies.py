"""Host arrays to and from the device, on the CPU (fake_hip): what is copied how,
and what happens where the library's staging buffer cannot be had."""
import pytest

import fake_hip

SETUP = """
ctx = wl.wl_create(0, 0x1000)
x = np.ones((512, 16), np.float32)
ens = wl.wl_ensemble_upload(ctx, x, x, 8)
fld = wl.field(1, 1.0, 1.0)
rho, T = np.linspace(0, 4, 3), np.geomspace(1e-2, 10, 7)
def average():
    return wl.wl_average_ex(ctx, ens, fld, rho, T, 1, wl.WL_FP64)
"""


@pytest.mark.parametrize("call,after", [("hostmalloc", 0), ("event", 0), ("event", 1)])
def test_staging_that_cannot_be_had(call, after):
    """A failure to make the staging buffer or either of its events: that call
    copies without it, a later one makes it, and all give the same."""
    fake_hip.run(SETUP + """
fake.fake_fail(%r, %d)
a = average()
assert any("pageable" in c for c in calls())
clear()
b = average()
assert any(c.startswith("h2d") and "pinned" in c for c in calls())
assert not any("pageable" in c for c in calls())
for k in wl.RESULT_KEYS:
    assert np.array_equal(a[k], b[k], equal_nan=True)
wl.wl_ensemble_free(ens)
wl.wl_destroy(ctx)
""" % (call.encode(), after))
