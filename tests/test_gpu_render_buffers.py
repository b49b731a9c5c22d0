"""What raster.render holds at a time: the image and its companions (20 bytes a pixel) take
the sort workspace's place, they do not come on top of it; and after an overflow the pair
count, which cannot change, is not read again."""
import pytest
import torch

from paper_2503_18402_amd import gsmi, raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("capacity", [2_000_000, 3_500_000])
@pytest.mark.parametrize("check", [True, False])
def test_image_takes_the_workspaces_place(capacity, check):
    sc, _ = scenes.small_scene()
    w, h = 1600, 1200
    cam = scenes.look_at((0, 0, -3.0), (0, 0, 0), w, h, 400.0)
    params = raster.to_device(sc)
    raster.render(params, [cam], capacity=capacity, check_capacity=check)
    torch.cuda.synchronize()
    base = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    fr = raster.render(params, [cam], capacity=capacity, check_capacity=check)
    peak = torch.cuda.max_memory_allocated() - base
    torch.cuda.synchronize()
    assert fr.capacity == capacity
    ws = gsmi.gs_bin_sort_workspace_bytes(1, fr.n, capacity)
    rest = gsmi.gs_proj_bytes(1, fr.n) + 4 * capacity + fr.ranges.numel() * 4
    assert peak <= max(ws, 20 * w * h) + rest + (4 << 20), peak  # (4 MiB: the allocator's rounding)


def test_count_is_read_once(monkeypatch):
    sc, cam = scenes.small_scene()
    params = raster.to_device(sc)
    reads = []
    wait = torch.cuda.Event.synchronize
    monkeypatch.setattr(torch.cuda.Event, "synchronize", lambda e: (reads.append(1), wait(e))[1])
    fr = raster.render(params, [cam], capacity=100)
    assert len(reads) == 1 and 100 < int(fr.n_pairs_dev.item()) <= fr.capacity
