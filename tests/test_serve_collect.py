"""Retirement in the serving loop: what a collection that fails leaves behind,
and which collections a backend is asked for."""
import pytest

from paper_1606_00310_amd.batch import Realization as R
from paper_1606_00310_amd.serve import BatchBackend, Request, Server

from test_serve_logic import Clock, FakeBackend


class Overflow(Exception):
    pass


class OneBadSlot(FakeBackend):
    """The sums of the realizations of one seed do not fit their type."""

    bad = 100

    def collect(self, slot):
        if self.used[slot][0].seed == self.bad:
            raise Overflow
        return super().collect(slot)


class OneBadSlotAtOnce(OneBadSlot):
    def collect_many(self, slots):
        for s in slots:
            yield self.collect(s)


@pytest.mark.parametrize("backend", [OneBadSlot, OneBadSlotAtOnce])
def test_a_failing_collection_fails_once(backend):
    """The error of one realization shows once; the others, those that finished
    in the same epoch among them, are served on."""
    be = backend(max_slots=8, budget=10**9)
    srv = Server(be, mcs_epoch=10, clock=Clock())
    for i in range(4):  # seeds 0, 100, 200, 300
        srv.submit(Request(i, [R(64, 64, 0.5, 0.0, 10, 100 * i)]))
    with pytest.raises(Overflow):
        srv.step()
    for i in range(4, 6):
        srv.submit(Request(i, [R(64, 64, 0.5, 0.0, 10, 100 * i)]))
    for _ in range(4):
        srv.step()
    assert [r.rid for r in srv.completed] == [0, 2, 3, 4, 5]
    assert set(srv.running) == {1}


class PlainBatch:
    """A batch with the calls that one collection at a time takes, and no other."""

    device = "cpu"

    def state(self, slot):
        import torch

        return torch.full((2, 2, 4, 1), slot), torch.tensor([7 * slot])

    def roughness(self, slot):
        return 16, slot, slot * slot, 0.5


@pytest.mark.parametrize("keep", [True, False])
def test_collects_from_a_batch_without_collect(keep):
    got = list(BatchBackend(PlainBatch(), keep_states=keep).collect_many([3, 5]))
    assert [(r["moments"], r["h0"]) for r in got] == [((16, 3, 9, 0.5), 21), ((16, 5, 25, 0.5), 35)]
    assert all(("slopes" in r) == keep for r in got)
