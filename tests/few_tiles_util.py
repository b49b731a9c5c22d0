"""Scenes for launches of few tiles: lists of about the same length in every tile."""
import numpy as np
import torch

from paper_2503_18402_amd import gsmi, raster, scenes

SPLAT = {8: 1.5, 16: 3.0}  # pixels


def even_scene(w, h, tile, length, seed=7):
    """Gaussians spread over a w x h view, about `length` in each tile's list."""
    rng = np.random.default_rng(seed)
    s, f = SPLAT[tile], float(w)
    tiles = -(-w // tile) * -(-h // tile)
    n = max(64, int(length * tiles / ((1 + 6 * s / tile) ** 2 * 0.8)))
    z = rng.uniform(-0.3, 0.3, n)
    d = 3.0 + z
    m = np.stack([(rng.uniform(0, w, n) - w / 2) / f * d, (rng.uniform(0, h, n) - h / 2) / f * d, z], 1)
    sc = dict(means=m, log_scales=np.log(3 * s / f) + rng.normal(0, 0.2, (n, 3)),
              quats=rng.normal(size=(n, 4)), opacity_logits=rng.normal(-1.0, 1, n),
              sh=np.concatenate([rng.normal(0.5, 0.2, (n, 1, 3)), rng.normal(0, 0.05, (n, 15, 3))], 1))
    return {k: v.astype(np.float32) for k, v in sc.items()}, scenes.look_at(
        (0, 0, -3.0), (0, 0, 0), w, h, f)


def step_kernel_us(w, h, tile, length, kernel, track_loss=True):
    """The least time of 5 x 20 steps that the kernels whose name holds `kernel` take a step."""
    sc, cam = even_scene(w, h, tile, length)
    pipe = raster.Pipeline(raster.to_device(sc), [cam], torch.rand(3 * w * h, device="cuda"),
                           tile=tile, lrs={k: 0.0 for k in raster.PARAM_NAMES})
    pipe.track_loss = track_loss
    for _ in range(10):
        pipe.step()
    best = float("inf")
    for _ in range(5):
        torch.cuda.synchronize()
        gsmi.gs_profile_enable(True)
        for _ in range(20):
            pipe.step()
        torch.cuda.synchronize()
        times = gsmi.gs_profile_collect()
        gsmi.gs_profile_enable(False)
        best = min(best, sum(t[1] for k, t in times.items() if kernel in k) / 20 * 1e3)
    return best
