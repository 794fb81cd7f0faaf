"""A freed ensemble's device memory goes to the next ensemble.  Work on another
stream than the context's (a captured launch replayed there, say) may still be
reading it: the free has to wait for the whole device, as hipFree does."""
import fake_hip


def test_free_waits_for_the_device_before_the_memory_is_kept():
    fake_hip.run("""
ctx = wl.wl_create(0, 0x1000)  # a stream of the caller
ens = wl.wl_ensemble_generate(ctx, 1, 0, 64, 256, 8)
fake.fake_foreign_work(1)
wl.wl_ensemble_free(ens)
assert not fake.fake_foreign_work_left()
clear()
ens = wl.wl_ensemble_generate(ctx, 1, 0, 64, 256, 8)
assert any("k_generate" in c for c in calls())
assert not any(c.startswith("malloc") for c in calls())  # the kept memory
wl.wl_ensemble_free(ens)
wl.wl_destroy(ctx)
assert fake.fake_used() == 0
""")
