"""What an epoch of an ensemble enqueues (no GPU)."""
from host_lib import host  # noqa: F401


def test_without_memory_for_teams_an_epoch_runs_without_them(host):
    """The messages of teams are allocated when a realization first wants one,
    perhaps with the device's memory full of states: the ensemble goes on."""
    host("""
e = Ensemble([(2048, 2048), (64, 64), (4096, 4096)])
fake.fake_fail_malloc(4 << 20)
log()
assert e.run(5) == 0 and [e.t(i) for i in range(3)] == [5, 5, 5]
lines = log()
assert [l.endswith("alone") for l in launches("onchip_kernel", lines)] == [True]   # the 64 x 64
assert lines.count("graph launch") == 1                                           # the others
fake.fake_fail_malloc(0)
assert e.run(5) == 0 and [e.t(i) for i in range(3)] == [10, 10, 10]
assert not [l for l in launches("onchip_kernel") if l.endswith("teams")]          # once is enough
e = Ensemble([(2048, 2048)])
assert e.run(5) == 0 and launches("onchip_kernel")[0].endswith("teams")
""")


def test_teams_that_do_not_form_have_a_list_of_their_own(host):
    """An epoch with teams carries, besides its lists, one for the persistent
    kernel that holds the teams' realizations too; that kernel is launched behind
    the teams either way."""
    host("""
sizes = [(64, 64), (2048, 2048), (8192, 8192), (4096, 4096)]
e = Ensemble(sizes, max_parts=4)
log()
assert e.run(7) == 0
lines = [l for l in log() if l.startswith(("launch", "graph"))]
assert [n for l in lines for n in ("onchip_reset", "onchip_kernel", "ensemble_kernel", "graph") if n in l] == [
    "onchip_reset", "onchip_kernel", "ensemble_kernel"]
assert lines[-2].endswith("teams") and lines[-1].endswith("behind teams")
assert fake.fake_items() == 4  # 8192 x 8192 in four parts; the others on chip
codes = [fake.fake_apart_order(k) for k in range(fake.fake_apart_items())]
assert {c & 0xfffff for c in codes} == {e.slots[i] for i in (1, 2, 3)}
for c in codes:  # every part of a split realization is there, with a geometry of its own
    s = c & 0xfffff
    assert sorted(x >> 20 for x in codes if x & 0xfffff == s) == list(range(fake.fake_apart_parts(s)))
    assert fake.fake_apart_depth(s) > 0
assert fake.fake_parts(e.slots[1]) > 1 and fake.fake_depth(e.slots[1]) == 0
""")


def test_many_small_states_share_a_compute_unit(host):
    """Workgroups of 256 threads run many small states side by side in LDS, as
    their configuration says; few of them, larger ones and other workgroups stay on chip."""
    host("""
def routes(n, X, Y, p, run=60, more=(), **config):
    e = Ensemble([(X, Y)] * n + list(more), n_mcs=10**6, p=p, **config)
    log()
    assert e.run(run) == 0
    lines = log()
    return len(launches("onchip_kernel", lines)), len([l for l in lines if l == "graph launch" or "ensemble_kernel" in l])

small = dict(block_threads=256, blocks_per_cu=8, lds_bytes=16384)
for p in (0.5, 0.9375, 1.0, 0.75):
    for X, Y in ((8, 8), (64, 64), (128, 128), (256, 256)):
        assert routes(2048, X, Y, p, **small)[0] == 0, (X, Y, p)
        assert routes(200, X, Y, p, **small) == (1, 0), (X, Y, p)
        assert routes(2048, X, Y, p) == (1, 0) and routes(2048, X, Y, p, block_threads=1024, blocks_per_cu=1) == (1, 0)
    assert routes(2048, 512, 512, p, **small) == (1, 0)
assert routes(2048, 64, 64, 0.5, lds_bytes=65536, block_threads=256, blocks_per_cu=1) == (1, 0)
# beside one that lasts longer than all of them on chip they cost nothing there
assert routes(300, 64, 64, 0.5, more=[(1024, 1024)], **small) == (1, 1) and fake.fake_items() == 0
assert routes(4000, 64, 64, 0.5, more=[(1024, 1024)], **small) == (1, 1) and fake.fake_items() == 4000
""")
