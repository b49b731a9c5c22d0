"""Empty tiles beside lists of the longest tier (more than 2048 keys): their ranges read
[0, 0), whichever block looks them up, and the long lists stay whole; with fewer tiles
than that tier's blocks, with several tiles a block, and without any long list.  Bit for
bit against the radix-sort binning of the same projected records."""
import numpy as np
import pytest
import torch

from paper_2503_18402_amd import gsmi, raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(100, 80), (520, 512), (1019, 1021)])  # 130, 4160, 16384 tiles
@pytest.mark.parametrize("heap", [1500, 2500, 9000])
def test_empty_tiles_beside_long_lists(w, h, heap):
    rng = np.random.default_rng(heap)
    cam = scenes.look_at((0, 0, -3.0), (0, 0, 0), w, h, 300.0)
    # three heaps that fall inside one tile each, in a view that is empty otherwise
    at = [(0.02, 0.02), (-0.3 * w / 300, 0.5 * h / 300), (w / 300 - 0.03, -h / 300 + 0.03)]
    m = np.concatenate([np.stack([np.full(heap, x), np.full(heap, y), rng.uniform(-0.5, 0.5, heap)], 1)
                        for x, y in at])
    n = len(m)
    m[:, :2] *= (3.0 + m[:, 2:]) / 3.0
    sc = dict(means=m, log_scales=np.full((n, 3), -7.0), quats=np.tile([1.0, 0, 0, 0], (n, 1)),
              opacity_logits=np.zeros(n), sh=np.zeros((n, 16, 3)))
    fr = raster.render(raster.to_device({k: v.astype(np.float32) for k, v in sc.items()}), [cam],
                       tile=8, want_keys=True)
    np_ = int(fr.n_pairs_dev.item())
    ws = torch.empty(gsmi.gs_bin_sort_radix_workspace_bytes(1, n, fr.capacity), dtype=torch.uint8,
                     device="cuda")
    keys, vals = torch.empty_like(fr.keys), torch.empty_like(fr.vals)
    ranges, npairs = torch.empty_like(fr.ranges), torch.zeros_like(fr.n_pairs_dev)
    gsmi.gs_bin_sort_radix(fr.cams_c, fr.cfg, n, fr.proj, fr.capacity, ws, keys, vals, ranges, npairs)
    torch.cuda.synchronize()
    r = ranges.view(-1, 2)
    length = r[:, 1] - r[:, 0]
    assert int(length.max()) >= heap and int((length == 0).sum()) >= length.numel() - 3 * 9
    assert torch.equal(fr.ranges, ranges)
    assert torch.equal(fr.keys[:np_], keys[:np_]) and torch.equal(fr.vals[:np_], vals[:np_])
