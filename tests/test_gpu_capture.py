"""Epochs of an ensemble under stream capture on the device's own runtime."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("X", [64, 2048])
def test_an_epoch_is_refused_under_capture(X):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_00310_amd import ScaError
    from paper_1606_00310_amd.batch import Batch, Realization, state_bytes

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        b = Batch(max_slots=1, arena_bytes=state_bytes(X, X), stream=stream)
        slots = b.admit([Realization(X, X, 0.5, 0.0, 100, 1)])
    torch.cuda.synchronize()
    with pytest.raises(ScaError):
        with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=stream):
            b.run(5)
    assert b.info(slots[0]).t == 0
    torch.cuda.synchronize()
