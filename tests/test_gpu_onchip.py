"""Ensemble realizations that stay on chip for an epoch, in one workgroup or in
a team of them, against their solo runs and the oracle, bit for bit."""
import sys

import numpy as np
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


def run_batch(reals, epochs=(), **config):
    from paper_1606_00310_amd.batch import Batch, state_bytes

    b = Batch(max_slots=len(reals), arena_bytes=sum(state_bytes(r.X, r.Y) for r in reals), config=config or None)
    slots = b.admit(reals)
    for e in epochs:
        b.run(e)
    while b.run(1 << 20):
        pass
    torch.cuda.synchronize()
    return b, slots


def check_solo(sca, b, slots, reals):
    for r, s in zip(reals, slots):
        lat = sca.Lattice(r.X, r.Y, seed=r.seed)
        lat.step(r.n_mcs, r.p, r.q, fuse=False)
        S, h0 = b.state(s)
        assert torch.equal(S, lat.slopes), r
        assert (b.info(s).t, int(h0[0])) == lat.meta(), r
        assert b.roughness(s) == lat.roughness(), r
        lat.close()
    b.close()


PROBS = [(0.5, 0.0), (0.5, 0.5), (0.75, 0.25), (0.9375, 0.0), (1.0, 0.0), (0.0, 1.0)]

# workgroups and rows per thread: partial words and idle waves; 2, 4 and 8 rows
# in one workgroup; teams of 2, 4 and 8 with 8 rows; the widest and the narrowest
# rows; too large for a team (128 MCS of 8192 x 2048 cost little), which the
# blocked passes take
SIZES = [(4, 4, 9), (16, 64, 9), (64, 64, 9), (128, 8, 9), (64, 2048, 7), (256, 256, 9), (512, 512, 7), (1024, 512, 7),
         (1024, 1024, 7), (128, 8192, 5), (2048, 1024, 7), (2048, 2048, 7), (4096, 2048, 5), (8192, 1024, 5),
         (8192, 128, 5), (512, 16384, 5), (8192, 2048, 3)]


@pytest.mark.parametrize("X,Y,n", SIZES)
def test_alone(sca, X, Y, n):
    """One realization at a time and probability pair: one workgroup, or one
    team with all its row groups at the edge of another's."""
    from paper_1606_00310_amd.batch import Realization as R

    for k, (p, q) in enumerate(PROBS):
        _say(f"[on chip] {X}x{Y} p={p} q={q}")
        reals = [R(X, Y, p, q, n, 50 + k)]
        b, slots = run_batch(reals, epochs=(1, 2))
        check_solo(sca, b, slots, reals)


def test_against_oracle(orc):
    from paper_1606_00310_amd.batch import Realization as R

    reals = [R(2048, 2048, 0.75, 0.25, 5, 1), R(2048, 2048, 0.5, 0.0, 6, 2), R(64, 128, 0.9375, 0.0, 40, 3),
             R(1024, 1024, 0.5, 0.5, 5, 4), R(32, 64, 0.5, 0.25, 30, 5)]
    b, slots = run_batch(reals)
    for r, s in zip(reals, slots):
        st = orc.flat(r.X, r.Y)
        orc.run(st, r.n_mcs, r.p, r.q, seed=r.seed)
        S, h0 = b.state(s)
        assert np.array_equal(S.cpu().numpy().view(np.uint64), orc.pack(st)), r
        assert int(h0[0]) == st.h0, r
    b.close()


def test_every_team_size_in_one_epoch(sca):
    """Long and short realizations for eight, four, two and one workgroups, more
    than there are teams, epochs of one MCS among them (a team may then be a
    realization ahead of its slowest member), beside per-site and oversized ones
    that the persistent kernel runs."""
    from paper_1606_00310_amd.batch import Realization as R

    reals = []
    for k in range(48):
        p, q = PROBS[k % len(PROBS)]
        reals.append(R(*[(4096, 2048), (2048, 2048), (2048, 1024), (1024, 1024), (64, 64), (4096, 1024)][k % 6], p, q,
                       1 + (7 * k) % 11, 900 + k))
    reals += [R(256, 256, 0.3, 0.1, 4, 77), R(8192, 2048, 0.5, 0.0, 3, 78), R(512, 64, 0.95, 0.0, 12, 79)]
    b, slots = run_batch(reals, epochs=(1, 1, 3))
    check_solo(sca, b, slots, reals)


def test_many_single_mcs_epochs(sca):
    """Teams of eight and four through a long list of one-MCS items, many
    launches in a row."""
    from paper_1606_00310_amd.batch import Realization as R

    reals = [R(2048, 2048, 0.5, 0.0, 12, 300 + k) for k in range(70)] + \
        [R(4096, 2048, 0.75, 0.0, 12, 400 + k) for k in range(40)]
    b, slots = run_batch(reals, epochs=(1,) * 12)
    check_solo(sca, b, [slots[i] for i in (0, 33, 69, 70, 109)], [reals[i] for i in (0, 33, 69, 70, 109)])


def test_two_batches_on_two_streams(sca):
    """Two ensembles with teams at once: the second waits for compute units, and
    both end with the bits of their solo runs."""
    from paper_1606_00310_amd.batch import Batch, Realization as R, state_bytes

    sets, batches = [], []
    for k in range(2):
        reals = [R(2048, 2048, 0.75, 0.25, 60, 10 * k + j) for j in range(6)] + [R(512, 512, 0.5, 0.0, 90, 70 + k)]
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            b = Batch(max_slots=len(reals), arena_bytes=sum(state_bytes(r.X, r.Y) for r in reals), stream=stream)
            slots = b.admit(reals)
        sets.append(reals)
        batches.append((b, slots))
    for _ in range(3):
        for b, _slots in batches:
            b.run(30)
    torch.cuda.synchronize()
    for (b, slots), reals in zip(batches, sets):
        check_solo(sca, b, slots, reals)


@pytest.mark.parametrize("n", [1, 32, 33])
def test_admission_initialises(sca, n):
    """Few states (launch argument) and many (staged table) start flat, whatever
    the arena held, one above 2^20 words among them."""
    from paper_1606_00310_amd import batch

    sizes = [(4, 4), (64, 64), (1024, 256), (8, 2048), (2048, 32768)]
    reals = [batch.Realization(*sizes[(i + 3 * (n == 1)) % len(sizes)], 0.5, 0.0, 3, i) for i in range(n)]
    b = batch.Batch(max_slots=n, arena_bytes=sum(batch.state_bytes(r.X, r.Y) for r in reals))
    b.arena.fill_(-1)
    for r, slot in zip(reals, b.admit(reals)):
        S, h0 = b.state(slot)
        W, nb = max(1, r.X // 128), min(64, r.X // 2)
        assert S.shape == (2, 2, r.Y, W) and int(h0[0]) == 0
        assert not S[:, 0].any() and bool((S[:, 1] == ((1 << nb) - 1 if nb < 64 else -1)).all())


@pytest.mark.parametrize("X,Y,p,q", [(2048, 2048, 0.75, 0.25), (4096, 1024, 0.5, 0.0), (64, 65536, 0.9375, 0.0),
                                     (8192, 512, 0.5, 0.5), (512, 8192, 0.5, 0.0)])
def test_teams_that_cannot_form(sca, X, Y, p, q):
    """A kernel on another stream keeps a compute unit from the launch: the
    realizations for teams run in memory, and later epochs make no teams."""
    from paper_1606_00310_amd.batch import Realization as R

    reals = [R(X, Y, p, q, 22, 5), R(128, 128, p, q, 22, 6), R(X, Y, 1.0, 0.0, 9, 7)]
    for _ in range(6):  # a stream may share the ensemble's hardware queue, and then delays it only
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.Stream()):
            torch.cuda._sleep(20_000_000)
        b, slots = run_batch(reals, epochs=(9, 5, 8))
        check_solo(sca, b, slots, reals)


@pytest.mark.parametrize("p,q", [(0.5, 0.0), (0.75, 0.25), (0.9375, 0.0), (1.0, 0.0)])
def test_teams_of_sixteen(sca, p, q):
    """Lattices that only sixteen workgroups hold, and ones that are split as far
    because little else runs."""
    from paper_1606_00310_amd.batch import Realization as R

    sizes = [(4096, 4096), (8192, 2048), (64, 131072), (2048, 8192), (2048, 2048), (512, 4096)]
    reals = [R(X, Y, p, q, 7 + 5 * (k % 3), 50 + k) for k, (X, Y) in enumerate(sizes)]
    b, slots = run_batch(reals, epochs=(1, 2, 8))
    check_solo(sca, b, slots, reals)
    reals = [R(2048, 2048, p, q, 33, 70)]
    b, slots = run_batch(reals)
    check_solo(sca, b, slots, reals)


@pytest.mark.parametrize("config", [dict(), dict(block_threads=1024, blocks_per_cu=1, depth=2, max_parts=4),
                                    dict(block_threads=512, blocks_per_cu=1, depth=4, max_parts=4),
                                    dict(block_threads=512, blocks_per_cu=1, depth=3, order=1)],
                         ids=["default", "split", "deep", "slot-order"])
def test_beside_blocked_passes(sca, config):
    """One epoch with realizations on chip, in teams, and ones that no team holds:
    blocked passes of the persistent kernel, split and whole, and per-site ones."""
    from paper_1606_00310_amd.batch import Realization as R

    reals = [R(8192, 4096, 0.5, 0.0, 7, 1), R(64, 64, 0.5, 0.0, 30, 2), R(8192, 8192, 0.75, 0.25, 5, 3),
             R(2048, 2048, 0.9375, 0.0, 9, 4), R(512, 512, 0.3, 0.1, 4, 5), R(1024, 131072, 0.5, 0.5, 4, 6),
             R(8192, 4096, 1.0, 0.0, 6, 7), R(256, 256, 0.625, 0.125, 11, 8)]
    b, slots = run_batch(reals, epochs=(3, 1), **config)
    check_solo(sca, b, slots, reals)
