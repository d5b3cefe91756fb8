"""Moments, two-time sums and heights against explicit heights: the sizes where
the split over words, rows and blocks changes, on rough surfaces and on the
steepest one."""
import sys

import numpy as np
import pytest

import lattice_util as U

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


def surface(X, Y, seed, steep=False):
    """h(x, y) = f(x) + g(y) with periodic bridges f and g, h = x + y mod 2."""
    rng = np.random.default_rng(seed)

    def bridge(n):
        e = np.repeat([1, -1], n // 2) if steep else rng.permutation(np.repeat([1, -1], n // 2))
        return np.cumsum(e) - e[0]

    h = bridge(Y)[:, None] + bridge(X)[None, :]
    if not steep:  # and some random moves, so that the rows differ
        for parity in (0, 1, 0, 1):
            h = U.height_rule_halfstep(h, parity, rng.random((Y, X)) < 0.7)
    return h


def snapshot(X, Y, h):
    """The surface in the packed layout: slopes, then h(0,0)."""
    sx, sy = U.slopes_from_heights(h)
    W, nb = max(1, X // 128), min(64, X // 2)
    out = np.zeros(4 * Y * W + 1, np.uint64)
    S = out[:-1].reshape(2, 2, Y, W)
    weights = np.uint64(1) << np.arange(nb, dtype=np.uint64)
    for d, s in ((0, sx), (1, sy)):
        for parity in (0, 1):
            for r in (0, 1):
                bits = s[r::2, (parity ^ r)::2].reshape(-1, W, nb).astype(np.uint64)
                S[d, parity, r::2] = (bits * weights).sum(-1, dtype=np.uint64)
    out[-1] = np.int64(h[0, 0]).astype(np.uint64)
    return torch.from_numpy(out.view(np.int64)).cuda()


# partial words, one word, every row width of one word per lane and several
# words per lane; one block of rows, few and (256) many, with and without rows
# to spare for the block's waves
SIZES = [(4, 4), (4, 1024), (8, 16), (16, 2048), (32, 4), (64, 256), (128, 128), (128, 4096), (256, 512), (512, 512),
         (1024, 1024), (2048, 16), (4096, 128), (8192, 64), (8192, 1024), (16384, 16), (32768, 32), (131072, 4),
         (64, 131072)]


@pytest.mark.parametrize("X,Y", SIZES)
@pytest.mark.parametrize("steep", [False, True])
def test_measurements(sca, X, Y, steep):
    _say(f"[measure] {X}x{Y} steep={steep}")
    ht, hs = surface(X, Y, 1, steep) - 12345 * 2, surface(X, Y, 2) + 2
    lat = sca.Lattice(X, Y, seed=1)
    old = snapshot(X, Y, hs)
    lat.restore(snapshot(X, Y, ht), 7)
    n = X * Y
    ht, hs = ht.astype(object) if n <= 4096 else ht.astype(np.int64), hs.astype(object) if n <= 4096 else hs.astype(np.int64)
    s1, s2 = int(ht.sum()), int((ht * ht).sum())
    ss, ts = int(hs.sum()), int((ht * hs).sum())
    assert lat.roughness() == (n, s1, s2, (n * s2 - s1 * s1) / (n * n))
    assert lat.autocorr(old) == (n, ts, s1, ss, (n * ts - s1 * ss) / (n * n))
    np.testing.assert_array_equal(lat.heights().cpu().numpy(), ht.astype(np.int32))
    # a window, into a buffer that is aligned to one int32 only
    from paper_1606_00310_amd import _lib as L

    y0, ny = Y // 4 + 1, max(1, Y // 2 - 1)
    buf = torch.full((ny * X + 6,), -7, dtype=torch.int32, device=lat.device)
    L.check(L.lib().sca_heights(lat._ctx, y0, ny, buf.data_ptr() + 4), "sca_heights")
    got = buf.cpu().numpy()
    np.testing.assert_array_equal(got[1:1 + ny * X].reshape(ny, X), ht[y0:y0 + ny].astype(np.int32))
    assert (got[:1] == -7).all() and (got[1 + ny * X:] == -7).all()


def test_many_contexts(sca):
    """More contexts than result slots: the rest reads back by copies."""
    lats = [sca.Lattice(8, 8, seed=i) for i in range(1030)]
    for lat in lats[-8:]:
        lat.step(3, 0.5, 0.0)
    for a, b in zip(lats[-8:-4], lats[-4:]):
        b.restore(a.snapshot(), 3)
        assert a.roughness() == b.roughness() and a.meta() == b.meta() and a.autocorr(b.snapshot())[0] == 64
        assert torch.equal(a.heights(), b.heights())
    for lat in lats:
        lat.close()
    lat = sca.Lattice(8, 8, seed=5)
    assert lat.roughness()[0] == 64


def test_collect_many(sca):
    """Moments and origin heights of more realizations than one launch takes,
    of one block and of several: as from one at a time."""
    from paper_1606_00310_amd import batch

    sizes = [(4, 4), (8, 64), (64, 32), (128, 128), (256, 512), (1024, 64), (4096, 4), (8192, 8), (8192, 4),
             (512, 2048), (8192, 64), (4, 8192)]
    reals = [batch.Realization(*sizes[i % len(sizes)], 0.75, 0.25 * (i % 2), 5 + i % 7, 1000 + i) for i in range(300)]
    b = batch.Batch(max_slots=len(reals), arena_bytes=sum(batch.state_bytes(r.X, r.Y) for r in reals))
    slots = b.admit(reals)
    while b.run(100):
        pass
    got = list(b.collect(slots[::-1]))[::-1]
    for s, (moments, h0) in zip(slots, got):
        assert moments == b.roughness(s) and h0 == int(b.state(s)[1][0])
    assert list(b.collect([])) == []
    b.release(slots[3])
    with pytest.raises(Exception):
        b.collect(slots[:5])
    assert next(b.collect(slots[:3])) == got[0]
