"""The backward blend of launches that the list-parallel kernel takes, at the tile counts
where its shape changes: a view alone (247 tiles, 16 waves a tile), and in batches of two
and three views (8 waves, which own several chunks of the long lists) and of seven (short
lists in blocks of their own), whose other views pass back nothing: the same gradients bit
for bit.  Then the times around these lines."""
import pytest
import torch

from paper_2503_18402_amd import raster, scenes
from tests.few_tiles_util import even_scene, step_kernel_us
from tests.test_gpu_blend_lists import _stack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,w,h", [(16, 300, 196), (8, 150, 98)])
@pytest.mark.parametrize("length,heap", [(6, 40), (47, 300), (47, 1100)])
def test_shapes_give_a_view_the_same_gradients(tile, w, h, length, heap):
    sc, cam = even_scene(w, h, tile, length)
    st = _stack(heap, "faint", seed=heap)
    params = raster.to_device({k: torch.cat([torch.from_numpy(sc[k]), torch.from_numpy(st[k])]).numpy()
                               for k in sc})
    up = torch.rand(3 * w * h, device="cuda", generator=torch.Generator("cuda").manual_seed(1)) - 0.5

    def grads(cams):
        fr = raster.render(params, cams, tile=tile)
        dL = torch.zeros_like(fr.image)
        dL[:3 * w * h] = up
        return fr, raster.render_backward(params, fr, dL)

    fr, want = grads([cam])
    deep = int(fr.last_contrib.max())
    assert deep > (0.9 * heap if heap > 48 else 0)
    for views in (2, 3, 7):
        _, got = grads([cam] + scenes.orbit_cameras(views - 1, 3.0, w, h, float(w)))
        torch.cuda.synchronize()
        for k in raster.PARAM_NAMES:
            assert torch.equal(got[k], want[k]), (views, k)


# 304 tiles of 16 against 256: 19% more work; a quarter is left for how the blocks fall on
# the CUs
@pytest.mark.parametrize("length", [10, 30, 100])
def test_more_tiles_than_wide_blocks_fit_do_not_queue(length):
    fits = step_kernel_us(256, 256, 16, length, "k_blend_bwd")
    more = step_kernel_us(304, 256, 16, length, "k_blend_bwd")
    assert more <= 1.5 * fits, (more, fits)


# 2000 tiles against 2050, where the ordinary kernel takes over: the same work but for 2.5%,
# and the launch's 2000 other blocks, which find their list short: 5 us for them, and a
# quarter for how the blocks fall on the CUs.
@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("length", [5, 10, 20])
def test_short_lists_take_no_longer_below_the_line(tile, length):
    k = 16 // tile
    few = step_kernel_us(800 // k, 640 // k, tile, length, "k_blend_bwd")
    many = step_kernel_us(800 // k, 656 // k, tile, length, "k_blend_bwd")
    assert few <= 1.25 * many + 5.0, (few, many)
