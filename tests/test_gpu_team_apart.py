"""Steps and epochs whose teams cannot form, since a kernel on another stream
holds a compute unit whole: that the fallback ran, and its bits."""
import sys
import time

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def sca():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1606_00310_amd as P

    P.lib()
    return P


class Holder:
    """Holds one compute unit for some 30 ms per call: an ensemble of one small
    per-site realization on a stream of its own, whose workgroup of 1024 threads
    takes all of the unit's registers; the kernel's other workgroups end at once."""

    def __init__(self):
        from paper_1606_00310_amd.batch import Batch, Realization, state_bytes

        self.stream = torch.cuda.Stream()
        with torch.cuda.stream(self.stream):
            self.batch = Batch(max_slots=1, arena_bytes=state_bytes(64, 64), stream=self.stream,
                               config=dict(block_threads=1024, blocks_per_cu=1, lds_bytes=65536, order=0,
                                           words_per_lane=1, depth=2, max_parts=1))
            self.batch.admit([Realization(64, 64, 0.3, 0.0, 10**9, 1)])
            self.batch.run(1)
        torch.cuda.synchronize()

    def hold(self):
        self.batch.run(3000)
        time.sleep(0.002)  # it runs


# rows and words per thread 2x1, 2x2, 4x1, 8x1 and 4x2; rows of 16 to 128 words
SHAPES = [(8192, 8192), (16384, 2048), (16384, 8192), (2048, 65536), (8192, 16384), (2048, 131072), (8192, 32768),
          (16384, 16384)]
PROBS = [(0.5, 0.0), (0.5, 0.5), (0.75, 0.25), (0.9375, 0.0), (0.625, 0.125), (1.0, 0.0)]


@pytest.mark.parametrize("X,Y", SHAPES)
@pytest.mark.parametrize("p,q", PROBS)
def test_lattice(sca, X, Y, p, q):
    """One pass pair with an MCS to spare, several, and one pass of a whole tile's depth."""
    ref = sca.Lattice(X, Y, seed=6)
    ns = [n for n in (2, 9, 64) if ref.plan(n, p, q)["kernel"].startswith("team_kernel")]
    if not ns:
        assert (X < 8192 or Y < 8192) or p == 1.0  # shapes that rarely go as teams
        pytest.skip("no team for this shape")
    for n in ns:
        for tries in range(8):  # a stream may share the lattice's hardware queue, and then delays it only
            holder = Holder()
            lat = sca.Lattice(X, Y, seed=6)
            lat.step(3, 0.75, 0.25, fuse=False)
            ref.reset()
            ref.step(3, 0.75, 0.25, fuse=False)
            torch.cuda.synchronize()
            _say(f"[apart] {X}x{Y} p={p} q={q} n={n} try {tries}")
            holder.hold()
            lat.step(n, p, q)
            torch.cuda.synchronize()
            ref.step(n, p, q, fuse=False)
            assert torch.equal(lat.slopes, ref.slopes) and lat.meta() == ref.meta()
            if not lat.plan(n, p, q)["kernel"].startswith("team_kernel"):
                break
        else:
            raise AssertionError("the team formed every time")


# rows of 1 to 64 words, realizations of two to sixteen workgroups, blocked passes
# for them (rows of 8 words and more) and none; a short one on chip beside them
ENSEMBLE = [(64, 65536), (128, 32768), (256, 16384), (512, 8192), (1024, 4096), (2048, 2048), (4096, 1024), (8192, 512),
            (4096, 4096), (8192, 2048)]


@pytest.mark.parametrize("X,Y", ENSEMBLE)
@pytest.mark.parametrize("config", [dict(), dict(block_threads=1024, blocks_per_cu=1, lds_bytes=65536, order=0,
                                                 words_per_lane=1, depth=2, max_parts=4),
                                    dict(block_threads=512, blocks_per_cu=1, depth=4, max_parts=2), dict(depth=0)],
                         ids=["default", "split", "deep", "unblocked"])
def test_ensemble(sca, X, Y, config):
    """All is made and the teams have formed once before the unit is held; then an
    epoch, whose teams cannot form, and one that goes without."""
    from paper_1606_00310_amd import lib
    from paper_1606_00310_amd.batch import Batch, Realization as R, state_bytes

    reals = [R(X, Y, 0.5, 0.0, 22, 5), R(X, Y, 0.75, 0.25, 22, 6), R(128, 128, 0.5, 0.0, 22, 7), R(X, Y, 1.0, 0.0, 9, 8),
             R(X, Y, 0.9375, 0.5, 22, 9)]
    for tries in range(8):  # a stream may share the ensemble's hardware queue, and then delays it only
        holder = Holder()
        b = Batch(max_slots=len(reals), arena_bytes=sum(state_bytes(r.X, r.Y) for r in reals), config=config)
        slots = b.admit(reals)
        b.run(4)
        torch.cuda.synchronize()
        assert lib().sca_debug_batch_teams(b._b) == 1
        _say(f"[apart] {X}x{Y} {config} try {tries}")
        holder.hold()
        b.run(9)
        torch.cuda.synchronize()
        apart = lib().sca_debug_batch_teams(b._b) == 0
        while b.run(1 << 20):
            pass
        for r, s in zip(reals, slots):
            lat = sca.Lattice(r.X, r.Y, seed=r.seed)
            lat.step(r.n_mcs, r.p, r.q, fuse=False)
            S, h0 = b.state(s)
            assert torch.equal(S, lat.slopes) and (b.info(s).t, int(h0[0])) == lat.meta(), r
            assert b.roughness(s) == lat.roughness(), r
        b.close()
        if apart:
            return
    raise AssertionError("the teams formed every time")


@pytest.mark.parametrize("X,Y", [(8192, 8192), (8192, 16384), (16384, 4096)])
@pytest.mark.parametrize("p,q", [(0.5, 0.0), (0.75, 0.25)])
@pytest.mark.parametrize("held", [False, True])
def test_a_step_of_two_launches(sca, X, Y, p, q, held):
    """513 MCS: a launch of as many as one takes, and one of a single MCS, whose
    band passes are a copy and an MCS."""
    lat, ref = sca.Lattice(X, Y, seed=8), sca.Lattice(X, Y, seed=8)
    for each in (lat, ref):
        each.step(3, 0.75, 0.25, fuse=False)
    assert lat.plan(513, p, q)["kernel"].startswith("team_kernel")
    holder = Holder()
    if held:
        holder.hold()
    lat.step(513, p, q)
    torch.cuda.synchronize()
    ref.step(513, p, q, fuse=False)
    assert torch.equal(lat.slopes, ref.slopes) and lat.meta() == ref.meta()
