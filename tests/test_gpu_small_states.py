"""Many small realizations in the LDS of workgroups of 256 threads, beside others
on chip and in teams: the bits of their solo runs."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PROBS = [(0.5, 0.0), (0.5, 0.5), (0.75, 0.25), (0.9375, 0.0), (1.0, 0.0), (0.0, 1.0), (0.625, 0.125)]
SIZES = [(4, 4), (8, 64), (64, 64), (64, 512), (128, 128), (256, 256), (512, 64), (1024, 64), (128, 4)]


@pytest.mark.parametrize("blocks,lds,words", [(8, 16384, 1), (2, 65536, 1), (4, 16384, 2)])
@pytest.mark.parametrize("more", [[], [(2048, 2048), (8192, 4096)]], ids=["alone", "beside"])
def test_against_solo_runs(blocks, lds, words, more):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1606_00310_amd as sca
    from paper_1606_00310_amd.batch import Batch, Realization as R, state_bytes

    reals = [R(*SIZES[i % len(SIZES)], *PROBS[i % len(PROBS)], 1 + i % 31, i) for i in range(3000)]
    reals += [R(X, Y, 0.5, 0.0, 5, 7) for X, Y in more]
    b = Batch(max_slots=len(reals), arena_bytes=sum(state_bytes(r.X, r.Y) for r in reals),
              config=dict(block_threads=256, blocks_per_cu=blocks, lds_bytes=lds, words_per_lane=words, max_parts=2))
    slots = b.admit(reals)
    for e in (3, 1, 1 << 20):
        b.run(e)
    torch.cuda.synchronize()
    for i in list(range(0, 3000, 47)) + list(range(3000, len(reals))):
        r, s = reals[i], slots[i]
        lat = sca.Lattice(r.X, r.Y, seed=r.seed)
        lat.step(r.n_mcs, r.p, r.q, fuse=False)
        S, h0 = b.state(s)
        assert torch.equal(S, lat.slopes) and (b.info(s).t, int(h0[0])) == lat.meta(), r
        lat.close()
    b.close()
