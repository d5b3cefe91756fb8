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

