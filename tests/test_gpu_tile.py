"""The on-chip tiles (all rows of a tile advanced together, in registers and
LDS) against the oracle from rough states, and the launch shapes that the cost
estimates choose against the two-launch form."""
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


def rough_pair(orc, sca, X, Y, seed):
    """The same rough surface (4 MCS at p = 3/4, q = 1/4) in the oracle and on the GPU."""
    st = orc.flat(X, Y, track_heights=False)
    orc.run(st, 4, 0.75, 0.25, seed=seed)
    S = np.ascontiguousarray(orc.pack(st)).reshape(-1).view(np.int64)
    lat = sca.Lattice(X, Y, seed=seed)
    lat.restore(torch.from_numpy(np.concatenate([S, np.array([st.h0], np.int64)])).to(lat.device), st.t)
    return st, lat


def detach_pass_buffer(lat):
    from paper_1606_00310_amd import _lib as L

    L.check(L.lib().sca_set_pass_buffer(lat._ctx, None, 0), "detach")


def assert_same(orc, lat, st):
    torch.cuda.synchronize()
    got, ref = lat.slopes.cpu().numpy().view(np.uint64), orc.pack(st)
    if not np.array_equal(got, ref):
        bad = np.argwhere(got != ref)
        raise AssertionError(f"{len(bad)} words differ, first at (d, pi, y, w) = {bad[0].tolist()}")
    assert lat.meta() == (st.t, st.h0)


# every draw class: odd and even numbers of draws, none; with and without removals
PROBS = [(0.5, 0.0), (0.5, 0.5), (0.75, 0.25), (0.9375, 0.0), (0.625, 0.125), (1.0, 0.0), (0.0, 1.0), (1.0, 1.0)]

# one workgroup: the smallest lattices (partial words, less than a wave), every
# row width of one word per lane, up to 1024 threads
WHOLE = [(4, 4), (8, 64), (64, 16), (64, 2048), (128, 128), (128, 2048), (256, 1024), (512, 512), (1024, 256),
         (2048, 8), (2048, 128), (4096, 4), (4096, 64)]


@pytest.mark.parametrize("X,Y", WHOLE)
@pytest.mark.parametrize("p,q", PROBS)
def test_whole_lattice(orc, sca, X, Y, p, q):
    _say(f"[whole] {X}x{Y} p={p} q={q}")
    st, lat = rough_pair(orc, sca, X, Y, seed=7 + X + Y)
    detach_pass_buffer(lat)  # one workgroup or half-step launches: no bands
    plan = lat.plan(6, p, q)
    assert plan["kernel"].startswith("tile_kernel") and plan["band"] == Y and plan["n_unfused"] == 0
    for n in (1, 6):
        lat.step(n, p, q)
        orc.run(st, n, p, q, seed=7 + X + Y)
        assert_same(orc, lat, st)


# bands: tiles of less than a wave, with idle lanes, taller than the lattice, of
# the most threads; odd depths (with four rows per thread the halo rounds up)
BANDS = [(64, 64, 3, 8), (128, 512, 4, 16), (256, 32, 13, 8), (512, 64, 5, 16), (1024, 128, 8, 32), (2048, 64, 7, 16),
         (2048, 256, 5, 128), (4096, 64, 8, 32), (4096, 64, 13, 16), (4096, 128, 3, 64)]


@pytest.mark.parametrize("X,Y,depth,band", BANDS)
@pytest.mark.parametrize("p,q", PROBS)
def test_bands(orc, sca, X, Y, depth, band, p, q):
    _say(f"[bands] {X}x{Y} depth={depth} band={band} p={p} q={q}")
    n = 2 * depth + 3
    st, lat = rough_pair(orc, sca, X, Y, seed=11 + X + depth)
    lat.set_blocking(depth, band)
    plan = lat.plan(n, p, q)
    assert plan["kernel"].startswith("tile_kernel") and (plan["n_pass"], plan["depth"], plan["band"]) == (2, depth, band)
    lat.step(n, p, q)
    orc.run(st, n, p, q, seed=11 + X + depth)
    assert_same(orc, lat, st)


@pytest.mark.parametrize("X,Y", [(512, 4096), (1024, 16384), (4096, 4096), (8192, 64), (8192, 2048), (16384, 128),
                                 (16384, 4096), (32768, 1024), (65536, 512), (65536, 4096)])
@pytest.mark.parametrize("p,q", [(0.5, 0.0), (0.75, 0.25), (1.0, 0.0), (0.93, 0.07)])
def test_automatic_shapes(sca, X, Y, p, q):
    """Whatever shape the cost estimates choose: the two-launch form's bits,
    for numbers of MCS with and without remainders, from a rough state."""
    a, b = sca.Lattice(X, Y, seed=5), sca.Lattice(X, Y, seed=5)
    for lat in (a, b):
        lat.step(3, 0.75, 0.25, fuse=False)
    for n in (1, 2, 5, 37):
        _say(f"[automatic] {X}x{Y} p={p} q={q} n={n}: {a.plan(n, p, q)}")
        a.step(n, p, q)
        b.step(n, p, q, fuse=False)
        assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()


# per-site words through LDS: words of one, two, four and eight bytes in use,
# whole lattices and bands up to the most words a tile holds, p below and at the
# ends of the threshold's range, dyadic values forced onto the path
PERSITE = [(4, 4, 0, 0), (16, 32, 0, 0), (32, 8, 0, 0), (64, 64, 0, 0), (128, 128, 0, 0), (512, 128, 0, 0),
           (2048, 64, 0, 0), (4096, 32, 0, 0), (32, 64, 3, 8), (128, 512, 5, 16), (256, 64, 4, 4), (1024, 256, 4, 4),
           (1024, 128, 8, 32), (2048, 64, 2, 8), (4096, 64, 4, 16), (4096, 128, 1, 4)]


@pytest.mark.parametrize("X,Y,depth,band", PERSITE)
@pytest.mark.parametrize("p,q", [(0.95, 0.0), (0.93, 0.07), (1.0 - 2.0**-33, 2.0**-40), (0.5, 0.25), (1.0, 0.3)])
def test_persite_tiles(orc, sca, X, Y, depth, band, p, q):
    _say(f"[per-site] {X}x{Y} depth={depth} band={band} p={p} q={q}")
    n = 2 * depth + 3
    st, lat = rough_pair(orc, sca, X, Y, seed=21 + X + depth)
    if depth:
        lat.set_blocking(depth, band)
    else:
        detach_pass_buffer(lat)
    plan = lat.plan(n, p, q, force_persite=True)
    assert "PerSite" in plan["kernel"] or Y * max(1, X // 128) > 256  # a large one may still go by half-steps
    lat.step(n, p, q, force_persite=True)
    orc.run(st, n, p, q, seed=21 + X + depth, force_persite=True)
    assert_same(orc, lat, st)


def test_without_pass_buffer(sca):
    """Narrow lattices never needed a pass buffer: they run without one."""
    for X, Y in ((128, 128), (4096, 512)):
        a, b = sca.Lattice(X, Y, seed=9), sca.Lattice(X, Y, seed=9)
        detach_pass_buffer(a)
        a.step(11, 0.5, 0.0)
        b.step(11, 0.5, 0.0)
        torch.cuda.synchronize()
        assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()


def test_graph_replays_of_tiles(sca):
    """The tiles inside one captured graph, with eager steps between."""
    for X, Y in ((128, 128), (2048, 1024)):
        a, b = sca.Lattice(X, Y, seed=3), sca.Lattice(X, Y, seed=3)
        for n in (9, 40, 9):
            a.step(n, 0.75, 0.25, graph=True)
            b.step(n, 0.75, 0.25, fuse=False)
            assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()
            a.step(3, 0.5, 0.0)
            b.step(3, 0.5, 0.0)
            assert torch.equal(a.slopes, b.slopes)


# words formed ahead: less than a wave of rows, one wave (two sets of producers
# with more than one draw), two to five waves; bands with idle lanes and with
# words outside the cone; up to 32 draws
AHEAD = [(4, 4, 0, 0), (32, 16, 0, 0), (128, 128, 0, 0), (256, 64, 0, 0), (64, 256, 0, 0), (1024, 64, 0, 0),
         (128, 512, 3, 4), (512, 128, 5, 8), (1024, 256, 6, 4), (2048, 64, 4, 4), (4096, 64, 3, 4), (4096, 32, 4, 4)]


@pytest.mark.parametrize("X,Y,depth,band", AHEAD)
@pytest.mark.parametrize("p,q", [(0.5, 0.0), (0.75, 0.25), (0.625, 0.0), (1.0, 0.5), (0.5 + 2.0**-11, 0.125),
                                 (1.0 - 2.0**-32, 2.0**-31)])
def test_words_ahead(orc, sca, X, Y, depth, band, p, q):
    _say(f"[ahead] {X}x{Y} depth={depth} band={band} p={p} q={q}")
    st, lat = rough_pair(orc, sca, X, Y, seed=31 + X + Y)
    if depth:
        lat.set_blocking(depth, band)
    else:
        detach_pass_buffer(lat)
    for n in (2 * max(depth, 3), 2 * depth + 7):  # from an even and an odd number of MCS
        # (with 32 draws, four waves of rows are slower than half-step launches)
        assert "Ahead" in lat.plan(n, p, q)["kernel"] or (depth == 0 and p > 0.99)
        lat.step(n, p, q)
        orc.run(st, n, p, q, seed=31 + X + Y)
        lat.step(1, p, q)
        orc.run(st, 1, p, q, seed=31 + X + Y)
        assert_same(orc, lat, st)


@pytest.mark.parametrize("X,Y", [(32768, 65536), (65536, 32768), (16384, 131072)])
@pytest.mark.parametrize("p,q", [(0.75, 0.25), (0.9375, 0.0)])
def test_full_height_bands_of_few_waves(sca, X, Y, p, q):
    """With fewer than four waves per SIMD at 128 rows the cost decides: 64 rows
    for these; the two-launch form's bits."""
    a, b = sca.Lattice(X, Y, seed=5), sca.Lattice(X, Y, seed=5)
    assert a.plan(33, p, q)["band"] == 64
    for n in (5, 33):
        _say(f"[few waves] {X}x{Y} p={p} q={q} n={n}: {a.plan(n, p, q)}")
        a.step(n, p, q)
        b.step(n, p, q, fuse=False)
        assert torch.equal(a.slopes, b.slopes) and a.meta() == b.meta()
