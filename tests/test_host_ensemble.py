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
