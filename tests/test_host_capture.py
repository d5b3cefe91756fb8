"""What calls do while their stream is being captured (no GPU)."""
from host_lib import host  # noqa: F401


def test_an_epoch_is_refused_under_capture(host):
    """An epoch stages its tables in host memory that the next one reuses, so a
    graph of it would replay whatever lies there: refused, as by the graph that
    every epoch used to launch."""
    host("""
for sizes in ([(64, 64)], [(2048, 2048)], [(8192, 8192)], [(64, 64), (2048, 2048)]):
    e = Ensemble(sizes)
    log()
    fake.fake_capturing(1)
    assert e.run(5) == L.SCA_EDEVICE and e.t(0) == 0
    assert not log()
    fake.fake_capturing(0)
    e = Ensemble(sizes)
    assert e.run(5) == 0 and e.t(0) == 5
    fake.fake_capturing(1)
    assert e.run(5) == L.SCA_EDEVICE and e.t(0) == 5
    fake.fake_capturing(0)
""")


def test_a_context_made_under_capture_has_no_teams(host):
    """The words of its teams would be cleared by the graph's launch, not before
    the next step."""
    host("""
fake.fake_capturing(1)
c = lattice(8192, 32768)
assert not launches("team_clear")
fake.fake_capturing(0)
assert lib.sca_step(c, 64, 0.5, 0.0) == 0 and not launches("team_kernel")
c = lattice(8192, 32768)
assert launches("team_clear")
assert lib.sca_step(c, 64, 0.5, 0.0) == 0 and launches("team_kernel")
""")
