"""raster.render under graph capture: refused where it would have to read the pair count
back, before anything is enqueued; captured and replayed where it does not."""
import pytest
import torch

from paper_2503_18402_amd import raster, scenes

pytestmark = pytest.mark.gpu


def test_reading_the_count_is_refused_under_capture():
    sc, cam = scenes.small_scene()
    params = raster.to_device(sc)
    x = torch.zeros(8, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x.add_(1.0)
        with pytest.raises(RuntimeError, match="capture"):
            raster.render(params, [cam])
    g.replay()  # the capture goes on
    torch.cuda.synchronize()
    assert x.eq(1.0).all()


def test_unread_count_is_captured():
    sc, cam = scenes.small_scene()
    params = raster.to_device(sc)
    want = raster.render(params, [cam])
    raster.render(params, [cam], capacity=want.capacity, check_capacity=False)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        got = raster.render(params, [cam], capacity=want.capacity, check_capacity=False)
    for _ in range(3):
        got.image.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got.image, want.image)
        assert int(got.n_pairs_dev.item()) == int(want.n_pairs_dev.item())
