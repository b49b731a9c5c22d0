"""raster.render on any stream the library's calls take: an object that has a stream handle
and is not torch's own stream class."""
from types import SimpleNamespace

import pytest
import torch

from paper_2503_18402_amd import raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("capacity", [100, None])
def test_stream_given_by_its_handle(capacity):
    sc, cam = scenes.small_scene()
    params = raster.to_device(sc)
    want = raster.render(params, [cam])
    own = torch.cuda.Stream()
    own.wait_stream(torch.cuda.current_stream())
    got = raster.render(params, [cam], capacity=capacity,
                        stream=SimpleNamespace(cuda_stream=own.cuda_stream))
    torch.cuda.synchronize()
    for k in ("image", "final_T", "last_contrib"):
        assert torch.equal(getattr(got, k), getattr(want, k)), k


@pytest.mark.parametrize("check", [True, False])
def test_count_is_not_cleared_behind_the_sort(check):
    """The current stream is busy while render runs on its own: nothing that it still has
    queued writes over the pair count."""
    sc, cam = scenes.small_scene()
    params = raster.to_device(sc)
    want = int(raster.render(params, [cam]).n_pairs_dev.item())
    own = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda._sleep(20_000_000)  # some milliseconds
    got = raster.render(params, [cam], capacity=200_000, check_capacity=check, stream=own)
    torch.cuda.synchronize()
    assert int(got.n_pairs_dev.item()) == want
