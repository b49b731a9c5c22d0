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
