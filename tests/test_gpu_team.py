"""One lattice in the registers of a team of workgroups: bit for bit the
two-launch form, whether the team forms or its workgroups work apart."""
import sys
import threading

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


def is_team(lat, n, p, q):
    return lat.plan(n, p, q)["kernel"].startswith("team_kernel")


# two, four and eight words per thread; rows of a quarter of a wave up to two
# words per lane; workgroups with idle waves and with all threads at work
SIZES = [(2048, 32768), (2048, 131072), (4096, 65536), (8192, 8192), (8192, 32768), (16384, 4096), (16384, 8192),
         (16384, 16384)]
PROBS = [(0.5, 0.0), (0.5, 0.5), (0.75, 0.25), (0.9375, 0.0), (0.625, 0.125), (1.0, 0.0), (1.0, 1.0)]


@pytest.mark.parametrize("X,Y", SIZES)
@pytest.mark.parametrize("p,q", PROBS)
def test_team(sca, X, Y, p, q):
    a, b = sca.Lattice(X, Y, seed=5), sca.Lattice(X, Y, seed=5)
    for lat in (a, b):
        lat.step(3, 0.75, 0.25, fuse=False)
    for n in (2, 9, 32):
        _say(f"[team] {X}x{Y} p={p} q={q} n={n}: {a.plan(n, p, q)['kernel']}")
        a.step(n, p, q)
        b.step(n, p, q, fuse=False)
        assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()
    assert is_team(a, 32, p, q) or X * Y < 1 << 28 or X < 8192 or p == 1.0


@pytest.mark.parametrize("X,Y", [(2048, 131072), (4096, 65536), (8192, 32768), (16384, 16384)])
@pytest.mark.parametrize("p,q", [(0.5, 0.0), (0.75, 0.25)])
def test_apart(sca, X, Y, p, q):
    """A kernel on another stream keeps a compute unit from the team, whose
    kernels of eight words per thread leave it no registers."""
    a, b = sca.Lattice(X, Y, seed=6), sca.Lattice(X, Y, seed=6)
    for lat in (a, b):
        lat.step(3, 0.75, 0.25, fuse=False)
    n = next(n for n in (64, 32, 16, 8, 4, 3, 2) if is_team(a, n, p, q))
    _say(f"[apart] {X}x{Y} p={p} q={q} n={n}")
    for _ in range(8):  # a stream may share the lattice's hardware queue, and then delays it only
        torch.cuda.synchronize()
        with torch.cuda.stream(torch.cuda.Stream()):
            torch.cuda._sleep(20_000_000)
        a.step(n, p, q)
        a.step(n, p, q)
        torch.cuda.synchronize()
        b.step(2 * n, p, q, fuse=False)
        assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()
        if not is_team(a, n, p, q):
            break
    assert not is_team(a, n, p, q)  # it could not form: no more teams here
    a.step(20, p, q)
    b.step(20, p, q, fuse=False)
    assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()


def test_threads_and_streams(sca):
    """Four lattices stepped by four threads, each on a stream of its own."""
    X, Y = 8192, 16384
    ref = sca.Lattice(X, Y, seed=7)
    ref.step(3, 0.75, 0.25, fuse=False)
    for n in (20, 33, 8):
        ref.step(n, 0.5, 0.0, fuse=False)
    torch.cuda.synchronize()
    lats = []

    def work():
        with torch.cuda.stream(torch.cuda.Stream()):
            lat = sca.Lattice(X, Y, seed=7)
            lat.step(3, 0.75, 0.25, fuse=False)
            for n in (20, 33, 8):
                lat.step(n, 0.5, 0.0)
            lats.append((lat, lat.meta()))

    threads = [threading.Thread(target=work) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert len(lats) == 4
    for lat, meta in lats:
        assert meta == ref.meta() and torch.equal(lat.slopes, ref.slopes)


def test_not_in_graphs(sca):
    """Steps that become part of a graph take the sweeps; eager ones between them the team."""
    X, Y = 8192, 32768
    a, b = sca.Lattice(X, Y, seed=8), sca.Lattice(X, Y, seed=8)
    for n in (20, 12, 20):
        a.step(n, 0.5, 0.0, graph=True)
        b.step(n, 0.5, 0.0, fuse=False)
        assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()
        assert is_team(a, n, 0.5, 0.0)
        a.step(n, 0.5, 0.0)
        b.step(n, 0.5, 0.0)
        assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()


def test_beside_an_ensemble(sca):
    """A lattice and an ensemble, both with teams, started together on two
    streams again and again: both end with the bits of the two-launch form."""
    from paper_1606_00310_amd.batch import Batch, Realization, state_bytes

    X, Y = 8192, 32768
    reals = [Realization(2048, 2048, 0.75, 0.25, 60, 10 + k) for k in range(6)] + [Realization(512, 512, 0.5, 0.0, 60, 3)]
    ref = sca.Lattice(X, Y, seed=9)
    ref.step(120, 0.5, 0.0, fuse=False)
    torch.cuda.synchronize()
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    for rep in range(3):
        _say(f"[beside] {rep}")
        with torch.cuda.stream(one):
            lat = sca.Lattice(X, Y, seed=9)
        with torch.cuda.stream(two):
            b = Batch(max_slots=len(reals), arena_bytes=sum(state_bytes(r.X, r.Y) for r in reals), stream=two)
            slots = b.admit(reals)
        torch.cuda.synchronize()
        for _ in range(6):
            with torch.cuda.stream(two):
                b.run(10)
            with torch.cuda.stream(one):
                lat.step(20, 0.5, 0.0)
        torch.cuda.synchronize()
        assert torch.equal(lat.slopes, ref.slopes) and lat.meta() == ref.meta()
        for r, s in zip(reals, slots):
            solo = sca.Lattice(r.X, r.Y, seed=r.seed)
            solo.step(r.n_mcs, r.p, r.q, fuse=False)
            assert torch.equal(b.state(s)[0], solo.slopes) and b.roughness(s) == solo.roughness()
        b.close()
