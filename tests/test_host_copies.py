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


PER_LOOP = """
ctx = wl.wl_create(0, 0x1000)
x = np.ones((512, 16), np.float32)
ens = wl.wl_ensemble_upload(ctx, x, x, 8)
fld = wl.field(0, 1.0, 1.0)
fake.fake_fill(1)  # fresh device memory holds 0, 1, 2, ...
def per_loop(side, out):
    rho, T = np.linspace(0, 4, side), np.geomspace(1e-2, 10, side)
    wl._check(wl._lib.wl_per_loop(ctx, ens, ctypes.byref(fld), wl._ptr(rho), side, wl._ptr(T),
                                  side, 0, wl.WL_FP32, 0, 512, *(wl._ptr(a) for a in out)), ctx)
    return out
def copied():
    return [int(c.split()[1]) for c in calls() if c.startswith("d2h")]
"""


@pytest.mark.parametrize("side", [1, 4, 8, 20, 33, 64])
def test_outputs_are_whole_and_nothing_else_is_copied(side):
    """Arrays of 4 KiB to 16 MiB each, pageable, pinned and mixed, with any of
    the three left out: the same values, and of the bytes that were not asked
    for at most a gap of 256 KiB."""
    fake_hip.run(PER_LOOP + """
import itertools
side = %d
n = 512 * side * side
full = per_loop(side, [np.zeros(n), np.zeros(n), np.zeros(n)])
assert full[0][0] == 0.0 and full[2][-1] == 3.0 * n - 1.0
for kinds in itertools.product((0, 1, 2), repeat=3):  # none, pageable, pinned
    out = [None if k == 0 else np.full(n, -1.0) if k == 1 else pinned(n) for k in kinds]
    clear()
    per_loop(side, out)
    for a, b in zip(out, full):
        assert a is None or np.array_equal(a, b), kinds
    asked = 8 * n * sum(k > 0 for k in kinds)
    assert asked <= sum(copied()) <= asked + (1 << 18), (kinds, copied())
    big = sum(k == 2 for k in kinds) if 8 * n >= 1 << 16 else 0
    # a pinned array of 64 KiB or more travels in one copy, however large
    assert copied()[:big] == [8 * n] * big, (kinds, copied())
""" % side)


@pytest.mark.parametrize("mib", [0.25, 7, 8, 9, 24])
def test_pinned_inputs_are_read_directly(mib):
    fake_hip.run("""
ctx = wl.wl_create(0, 0x1000)
n = int(%r * 131072)
for a, direct in ((pinned(n), True), (np.zeros(n), False)):
    a[:] = np.arange(n)
    out = np.zeros((16, 16))
    clear()
    wl._check(wl._lib.wl_correlation(ctx, a.ctypes.data, n // 16, 16, 0, out.ctypes.data), ctx)
    sizes = [int(c.split()[1]) for c in calls() if c.startswith("h2d")]
    assert all("pinned" in c for c in calls() if c.startswith("h2d"))
    assert sum(sizes) == 8 * n
    assert len(sizes) == (1 if direct else -(-8 * n // (8 << 20)))
""" % mib)
