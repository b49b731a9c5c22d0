"""The binning's blocks at their edges, bit for bit against the radix-sort binning of
the same projected records: one item, one more than a block's, several rounds per
block and more blocks than their positions are added up for directly; views of
few and of many tiles in one launch, in any order; footprints of every tile of a
view next to ones of a single tile; both storage orders; and the one-kernel binning of
small launches up to its limits, with a capacity that just fits and one that does not."""
import numpy as np
import pytest
import torch

from paper_2503_18402_amd import gsmi, raster, scenes

pytestmark = pytest.mark.gpu


def _cams(sizes):
    cams = scenes.orbit_cameras(len(sizes), 3.0, 64, 64, 60.0)
    return [scenes.Camera(**{**c.__dict__, "width": w, "height": h, "cx": w / 2, "cy": h / 2,
                             "fx": 0.9 * w, "fy": 0.9 * w}) for c, (w, h) in zip(cams, sizes)]


SMALL, FEW, MANY = (40, 24), (300, 200), (1019, 525)


@pytest.mark.parametrize("n,sizes,tile,giants,spatial", [
    (1, [SMALL, MANY], 8, 0, False),
    (1, [SMALL], 16, 1, False),
    (1023, [SMALL, FEW, SMALL], 8, 3, False),
    (1025, [(47, 33)] * 7, 8, 1, True),
    (8192, [FEW], 16, 4, False),
    (8193, [FEW], 16, 4, False),
    (2048, [(256, 250), (8, 8)] * 2, 8, 0, False),
    (257, [MANY] * 3, 16, 2, False),
    (1025, [SMALL, MANY, FEW], 8, 5, False),
    (2049, [FEW, SMALL] * 8, 16, 0, True),
    (600_001, [MANY, SMALL, FEW], 16, 3, True),
    (300_001, [SMALL] * 9 + [MANY] + [FEW] * 6, 16, 1, False),
])
def test_blocks_equal_radix(n, sizes, tile, giants, spatial):
    sc = scenes.make_scene(n, seed=n, ls_mu=-5.0, ls_sigma=0.3)
    sc["log_scales"][:giants] = 1.0
    if spatial:
        o = np.lexsort((sc["means"][:, 0] // 0.2, sc["means"][:, 1] // 0.2, sc["means"][:, 2] // 0.2))
        sc = scenes.subset(sc, o)
    cams = _cams(sizes)
    fr = raster.render(raster.to_device(sc, "cuda"), cams, tile=tile, want_keys=True)
    np_ = int(fr.n_pairs_dev.item())
    assert np_ <= fr.capacity
    proj = fr.proj.clone()
    ws = torch.empty(max(gsmi.gs_bin_sort_radix_workspace_bytes(len(cams), n, fr.capacity), 16),
                     dtype=torch.uint8, device="cuda")
    keys, vals = torch.empty_like(fr.keys), torch.empty_like(fr.vals)
    ranges, npairs = torch.empty_like(fr.ranges), torch.zeros_like(fr.n_pairs_dev)
    gsmi.gs_bin_sort_radix(fr.cams_c, fr.cfg, n, fr.proj, fr.capacity, ws, keys, vals, ranges,
                           npairs)
    torch.cuda.synchronize()
    assert int(npairs.item()) == np_ and np_ > 0
    assert torch.equal(keys[:np_], fr.keys[:np_])
    assert torch.equal(vals[:np_], fr.vals[:np_])
    assert torch.equal(ranges, fr.ranges)
    assert torch.equal(proj, fr.proj)   # the items' pair offsets and the total


@pytest.mark.parametrize("n", [700, 9000])
def test_capacity_that_just_fits(n):
    sc = scenes.make_scene(n, seed=n, ls_mu=-3.0)
    cams = _cams([FEW, SMALL])
    params = raster.to_device(sc, "cuda")
    want = raster.render(params, cams, tile=16)
    total = int(want.n_pairs_dev.item())
    fits = raster.render(params, cams, tile=16, capacity=total, check_capacity=False)
    over = raster.render(params, cams, tile=16, capacity=total - 1, check_capacity=False)
    torch.cuda.synchronize()
    assert int(fits.n_pairs_dev.item()) == int(over.n_pairs_dev.item()) == total
    assert torch.equal(fits.ranges, want.ranges) and torch.equal(fits.vals, want.vals[:total])
    assert not over.ranges.any()
