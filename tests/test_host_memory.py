"""Device memory that the contexts hold unused, on the CPU (fake_hip): it goes
back before an allocation of any of them fails, and freed ensembles' memory is
kept only while much more is free."""
import fake_hip


def test_idle_memory_of_every_context_serves_an_allocation():
    fake_hip.run("""
a, b = wl.wl_create(0, 0x1000), wl.wl_create(0, 0x1000)
def ens(ctx, loops):
    return wl.wl_ensemble_generate(ctx, 1, 0, loops, 1024, 8)
wl.wl_ensemble_free(ens(a, 1024))          # 24 MiB kept by a
wl.wl_correlation(a, np.ones((2, 2048)))   # its scratch kept by a
mib = 1 << 20
held = fake.fake_used()
assert held > 24 * mib
# what is left does not hold 36 MiB without a's ensemble block ...
fake.fake_limit(held + 20 * mib)
e = ens(b, 1536)
wl.wl_ensemble_free(e)
# ... nor what remains without the scratch that a does not work with
wl.wl_correlation(a, np.ones((2, 2048)))
held = fake.fake_used()
fake.fake_limit(held + 20 * mib)
e = ens(b, 1536)
wl.wl_ensemble_free(e)
fake.fake_limit(1 << 38)
wl.wl_correlation(a, np.ones((2, 2048)))   # and a makes it again
wl.wl_destroy(a)
wl.wl_destroy(b)
assert fake.fake_used() == 0
""")


def test_scratch_in_use_stays():
    """The call that allocates keeps the scratch it works with, and fails
    cleanly when nothing else can go."""
    fake_hip.run("""
a = wl.wl_create(0, 0x1000)
wl.wl_correlation(a, np.ones((2, 512)))
fake.fake_limit(fake.fake_used())
wl.wl_correlation(a, np.ones((2, 512)))
try:
    wl.wl_correlation(a, np.ones((2, 4096)))
except wl.WLError as e:
    assert e.code == wl.WL_ENOMEM, e
else:
    raise AssertionError("no room, no error")
fake.fake_limit(1 << 38)
wl.wl_correlation(a, np.ones((2, 4096)))
wl.wl_destroy(a)
assert fake.fake_used() == 0
""")


def test_freed_ensembles_are_kept_while_memory_is_plentiful():
    fake_hip.run("""
mib = 1 << 20
a = wl.wl_create(0, 0x1000)
def ens(loops):
    return wl.wl_ensemble_generate(a, 1, 0, loops, 1024, 8)
base = fake.fake_used()
fake.fake_limit(base + 1600 * mib)
e = ens(8192)                               # 192 MiB
wl.wl_ensemble_free(e)                      # 1400 free: kept
assert fake.fake_used() - base > 192 * mib
e = ens(8192)
assert fake.fake_used() - base < 193 * mib  # reused
fake.fake_limit(fake.fake_used() + 700 * mib)
wl.wl_ensemble_free(e)                      # less than four times as much free
assert fake.fake_used() == base
# the smallest block that fits is taken
fake.fake_limit(1 << 38)
big, small = ens(1304), ens(1104)
wl.wl_ensemble_free(big)
wl.wl_ensemble_free(small)
e = ens(1056)
assert fake.fake_used() - base < 57 * mib
f = ens(1256)
assert fake.fake_used() - base < 57 * mib   # the larger one served it
wl.wl_ensemble_free(e)
wl.wl_ensemble_free(f)
wl.wl_destroy(a)
assert fake.fake_used() == 0
""")
