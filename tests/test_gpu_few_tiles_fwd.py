"""The forward blend of launches that the list-parallel kernel takes: its shapes (a block
per 8x8 group of a tile, or one per tile) give one view the same bits, short lists and
long ones side by side; and lists that are not long take no longer just below the tile
count from which the ordinary kernel takes over than just above it."""
import pytest
import torch

from paper_2503_18402_amd import raster, scenes
from tests.few_tiles_util import even_scene, step_kernel_us
from tests.test_gpu_blend_lists import _stack

pytestmark = pytest.mark.gpu


def _scene(w, h, tile, length, heap):
    sc, cam = even_scene(w, h, tile, length)
    st = _stack(heap, "faint", seed=heap)
    both = {k: torch.cat([torch.from_numpy(sc[k]), torch.from_numpy(st[k])]).numpy() for k in sc}
    return both, cam


@pytest.mark.parametrize("tile,w,h,views", [(16, 300, 196, (3, 4, 7)), (8, 150, 98, (3, 7))])
@pytest.mark.parametrize("length,heap", [(6, 40), (47, 1100)])
def test_shapes_give_a_view_the_same_bits(tile, w, h, views, length, heap):
    """One view alone (247 tiles), and in a batch of 741, 988 or 1729."""
    sc, cam = _scene(w, h, tile, length, heap)
    params = raster.to_device(sc)
    want = raster.render(params, [cam], tile=tile)
    n = w * h
    ln = (want.ranges.view(-1, 2)[:, 1] - want.ranges.view(-1, 2)[:, 0])
    assert int(ln.min()) <= 48 and (heap < 48 or int(ln.max()) > 1024)
    for nv in views:
        more = scenes.orbit_cameras(nv - 1, 3.0, w, h, float(w))
        got = raster.render(params, [cam] + more, tile=tile)
        torch.cuda.synchronize()
        assert torch.equal(got.image[:3 * n], want.image)
        assert torch.equal(got.final_T[:n], want.final_T)
        assert torch.equal(got.last_contrib[:n], want.last_contrib)


# 2000 tiles against 2050: the same work but for 2.5%; half again is left for how the
# blocks fall on the CUs
@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("length", [5, 10, 30])
@pytest.mark.parametrize("track_loss", [True, False])
def test_short_lists_take_no_longer_below_the_line(tile, length, track_loss):
    k = 16 // tile
    few = step_kernel_us(800 // k, 640 // k, tile, length, "k_blend_fwd", track_loss)
    many = step_kernel_us(800 // k, 656 // k, tile, length, "k_blend_fwd", track_loss)
    assert few <= 1.5 * many, (few, many)
