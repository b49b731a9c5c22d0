"""Lists whose depths are all equal go to the 64-bit networks at once, bit for bit as the
radix sort has them; lists of few distinct depths, which either way may take, too."""
import numpy as np
import pytest
import torch

from paper_2503_18402_amd import gsmi, raster, scenes

pytestmark = pytest.mark.gpu


def _frame(n, depths, w, h, seed=3):
    """Small Gaussians over a view whose depths take `depths` values (0: all differ)."""
    rng = np.random.default_rng(seed)
    cam = scenes.look_at((0, 0, 0), (0, 0, 1), w, h, float(w))
    z = rng.choice(np.linspace(2.0, 3.0, depths), n) if depths else rng.uniform(2, 3, n)
    m = np.stack([rng.uniform(-0.5, 0.5, n) * z, rng.uniform(-0.5, 0.5, n) * h / w * z, z], 1)
    sc = dict(means=m, log_scales=np.full((n, 3), np.log(2.0 * 2.5 / w)),
              quats=np.tile([1.0, 0, 0, 0], (n, 1)), opacity_logits=np.zeros(n),
              sh=np.zeros((n, 16, 3)))
    return raster.render(raster.to_device({k: v.astype(np.float32) for k, v in sc.items()}), [cam],
                         want_keys=True)


def _sort(fr, ws, keys=None):
    gsmi.gs_bin_sort(fr.cams_c, fr.cfg, fr.n, fr.proj, fr.capacity, ws, keys, fr.vals, fr.ranges,
                     fr.n_pairs_dev)


@pytest.mark.parametrize("n", [3_000, 60_000, 250_000, 1_000_000])  # lists of 4 to 1200
@pytest.mark.parametrize("depths", [1, 2, 20, 60])
def test_few_depths_equal_radix(n, depths):
    fr = _frame(n, depths, 800, 656)
    np_ = int(fr.n_pairs_dev.item())
    assert n <= np_ <= fr.capacity
    ws = torch.empty(gsmi.gs_bin_sort_radix_workspace_bytes(1, n, fr.capacity), dtype=torch.uint8,
                     device="cuda")
    keys, vals = torch.empty_like(fr.keys), torch.empty_like(fr.vals)
    ranges, npairs = torch.empty_like(fr.ranges), torch.zeros_like(fr.n_pairs_dev)
    gsmi.gs_bin_sort_radix(fr.cams_c, fr.cfg, n, fr.proj, fr.capacity, ws, keys, vals, ranges, npairs)
    torch.cuda.synchronize()
    assert torch.equal(fr.ranges, ranges)
    assert torch.equal(fr.keys[:np_], keys[:np_]) and torch.equal(fr.vals[:np_], vals[:np_])


def test_equal_depths_cost_the_networks_alone():
    """A network on 64-bit keys takes about twice as long as one on words (a compare and four
    selects a comparator against a minimum and a maximum); the words, the exchange passes and
    then the network take over three times as long."""
    times = []
    for depths in (0, 1):
        fr = _frame(400_000, depths, 1600, 1064)
        ws = torch.empty(gsmi.gs_bin_sort_workspace_bytes(1, fr.n, fr.capacity), dtype=torch.uint8,
                         device="cuda")
        for _ in range(5):
            _sort(fr, ws)
        best = float("inf")
        for _ in range(5):
            torch.cuda.synchronize()
            gsmi.gs_profile_enable(True)
            for _ in range(10):
                _sort(fr, ws)
            torch.cuda.synchronize()
            t = gsmi.gs_profile_collect()
            gsmi.gs_profile_enable(False)
            best = min(best, t["k_tile_sort_wave"][1] / 10 * 1e3)
        times.append(best)
    assert times[1] <= 2.6 * times[0], times
