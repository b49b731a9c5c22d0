"""The per-tile sorts on 32-bit words against the radix sort of the same pairs, bit for
bit: list lengths at the edges of every tier and of a lane's and a wave's keys; depths
that spread over one binade, over twenty-four (a word holds few of their bits), that
come in pairs, in runs longer than the exchange passes put right, and that are all equal;
alone, and with as many Gaussians behind the camera as the one-kernel binning takes."""
import numpy as np
import pytest
import torch

from paper_2503_18402_amd import gsmi, raster, scenes

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 8, 9, 63, 65, 255, 257, 511, 512, 513, 1023, 1025, 2047, 2048, 2049, 4097, 8191,
          8192, 8193, 16385]


@pytest.mark.parametrize("behind", [0, 8192])
@pytest.mark.parametrize("depths", ["binade", "wide", "pairs", "runs", "equal"])
def test_word_sorts_equal_radix(depths, behind):
    rng = np.random.default_rng(len(depths))
    cam = scenes.look_at((0, 0, 0), (0, 0, 1), 16, 16, 20.0)
    for n in COUNTS:
        z = {"binade": lambda: rng.uniform(1, 2, n), "wide": lambda: 2.0 ** rng.uniform(-1, 23, n),
             "pairs": lambda: np.repeat(rng.uniform(1, 5, (n + 1) // 2), 2)[:n],
             "runs": lambda: np.repeat(rng.uniform(1, 5, n // 40 + 1), 40)[:n],
             "equal": lambda: np.full(n, 1.5)}[depths]().astype(np.float32)
        rng.shuffle(z)
        ls = np.log(0.3 * z)[:, None] + np.zeros((1, 3))
        z, ls = np.concatenate([z, np.full(behind, -3.0)]), np.concatenate([ls, np.zeros((behind, 3))])
        N = n + behind
        sc = dict(means=np.stack([0 * z, 0 * z, z], 1), log_scales=ls,
                  quats=np.tile([1.0, 0, 0, 0], (N, 1)), opacity_logits=np.zeros(N),
                  sh=np.zeros((N, 16, 3)))
        sc = {k: v.astype(np.float32) for k, v in sc.items()}
        fr = raster.render(raster.to_device(sc), [cam], tile=16, want_keys=True)
        assert int(fr.n_pairs_dev.item()) == n
        ws = torch.empty(gsmi.gs_bin_sort_radix_workspace_bytes(1, N, fr.capacity),
                         dtype=torch.uint8, device="cuda")
        keys, vals = torch.empty_like(fr.keys), torch.empty_like(fr.vals)
        ranges, npairs = torch.empty_like(fr.ranges), torch.zeros_like(fr.n_pairs_dev)
        gsmi.gs_bin_sort_radix(fr.cams_c, fr.cfg, N, fr.proj, fr.capacity, ws, keys, vals, ranges,
                               npairs)
        torch.cuda.synchronize()
        assert torch.equal(keys[:n], fr.keys[:n]) and torch.equal(vals[:n], fr.vals[:n]), n
        assert torch.equal(ranges, fr.ranges), n
