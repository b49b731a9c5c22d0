"""The blend kernels at the edges of their chunks, against the FP64 oracle: lists of
one entry, of the 64 a chunk holds and one to either side of one and two chunks,
and what is left for the last flush of the backward's sums; records that may
reach the opacity clamp among plain ones; tiles of 8, 16 and 32 pixels, ragged views.
The views have more tiles than the list-parallel kernels take, so every list is walked by
the ordinary ones.  Then the list-parallel kernels on a small view: one chunk, chunks of the least size, the last of one round
and the first of the next, a wave's second batch, with pixels that stop and that do not.

Tolerances: an image value sums at most 129 weighted colours in float32 (below
129 * 2^-24 = 8e-6); T is recovered over at most 129 divisions, each within 2^-22,
so a term of a gradient carries about 129^0.5 * 2^-22 = 2.7e-6 of itself: below the
1e-5 of the terms' scale that check_grads allows beside 1e-3 of the result.  (The
small view: at most 1025 entries, whose roundings of T add up to 1025^0.5 * 2^-24 =
2e-6, and at most 1025 / 8 divisions.)"""
import numpy as np
import pytest
import torch

from oracle import project, render
from paper_2503_18402_amd import raster, scenes
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

SIZES = {8: (507, 261), 16: (1019, 525), 32: (205, 119)}  # 64 x 33 tiles (32: no list-parallel form)


def _stack(count, kind, seed):
    """`count` Gaussians a few pixels wide around the view's centre, front to back."""
    rng = np.random.default_rng(seed)
    m = np.zeros((count, 3))
    m[:, :2] = rng.normal(0, 0.02, (count, 2))
    m[:, 2] = rng.permutation(np.linspace(-0.5, 0.5, count)) if count > 1 else 0.0
    s = rng.normal(-3.6, 0.2, (count, 3))
    q = rng.normal(size=(count, 4))
    o = rng.uniform(-3.6, -2.6, count)
    if kind == "faint":  # no pixel stops
        o = rng.uniform(-5.0, -4.5, count)
    if kind == "dense":  # every box holds the centre
        m[:, :2] *= 0.25
    front = np.argsort(m[:, 2])
    if kind == "clamped":  # the last and the one at two thirds may reach 0.99
        o[front[[-1, (2 * count) // 3]]] = 7.0
    d = dict(means=m, log_scales=s, quats=q, opacity_logits=o,
             sh=np.concatenate([rng.normal(0.5, 0.2, (count, 1, 3)),
                                rng.normal(0, 0.05, (count, 15, 3))], 1))
    return {k: v.astype(np.float32) for k, v in d.items()}


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("count,kind", [(1, "plain"), (63, "plain"), (64, "clamped"),
                                        (65, "plain"), (66, "plain"), (128, "plain"),
                                        (129, "clamped")])
def test_lists_at_chunk_edges_match_oracle(tile, count, kind):
    _compare(*SIZES[tile], tile, count, kind, least=0.9)


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("count,kind", [(1, "plain"), (24, "plain"), (25, "clamped"),
                                        (48, "plain"), (49, "plain"), (384, "faint"),
                                        (385, "clamped"), (769, "faint"), (1025, "faint"),
                                        (384, "dense"), (385, "dense")])
def test_lists_of_few_tiles_match_oracle(tile, count, kind):
    _compare(61, 45, tile, count, kind, least=0.5)


def _compare(w, h, tile, count, kind, least):
    cam = scenes.look_at((0, 0, -3.0), (0, 0, 0), w, h, 300.0)
    sc = _stack(count, kind, seed=count)
    P = project.project(sc, cam, tile=tile)
    if kind in ("plain", "dense"):
        assert max(map(len, render.tile_candidates(P))) == count
    ys, xs = np.mgrid[h // 2 - 22:h // 2 + 23, w // 2 - 22:w // 2 + 23]
    pix = (ys * w + xs).ravel()
    F = render.render_fwd(P, pixels=pix)
    if kind == "faint":
        assert F["final_T"].min() > 2e-4
    up = U.zero_flagged(np.random.default_rng(9).uniform(-1, 1, (3, len(pix))), F)
    full = np.zeros((3, w * h), np.float32)
    full[:, pix] = up
    _, frame, g = U.run(sc, [cam], tile=tile, lds_batch=128, upstream=[full], want_keys=False)
    img = frame.image.view(3, -1).cpu().numpy()[:, pix]
    ok = ~F["flag"]
    assert ok.mean() > least
    assert np.abs(img - F["image"])[:, ok].max() < 1e-5
    B = render.render_bwd(sc, P, up, pixels=pix, with_bound=True)
    keep = ~U.gaussian_flags(P)
    for name in raster.PARAM_NAMES:
        U.check_grads(g[name], B["d_" + name], B["bound"]["d_" + name], mask=keep, name=name,
                      max_frac=1.0)


@pytest.mark.parametrize("tile", [8, 16, 32])
def test_plain_and_general_walks_agree(tile):
    """One opaque Gaussian of a few pixels, behind the others, sends the lists it joins
    to the general walk: every pixel it does not reach keeps its bits."""
    w, h = SIZES[tile]
    cam = scenes.look_at((0, 0, -3.0), (0, 0, 0), w, h, 300.0)
    sc = _stack(60, "plain", seed=5)
    one = {k: v[:1].copy() for k, v in sc.items()}
    one["means"][0] = (0.03, 0.02, 0.9)
    one["log_scales"][0], one["opacity_logits"][0] = -5.5, 7.0
    both = {k: np.concatenate([sc[k], one[k]]) for k in sc}
    _, fa, _ = U.run(sc, [cam], tile=tile, want_keys=False)
    _, fb, _ = U.run(both, [cam], tile=tile, want_keys=False)
    d = fa.last_contrib != fb.last_contrib
    P = project.project(both, cam, tile=tile)
    B = render.render_fwd(P, pixels=np.nonzero(d.cpu().numpy().ravel())[0])
    assert 4 <= len(B["pixels"]) <= 200 and (B["last_id"][~B["flag"]] == 60).all()
    same = torch.ones(w * h, dtype=torch.bool, device="cuda")
    same[torch.from_numpy(B["pixels"]).cuda()] = False
    assert torch.equal(fa.image.view(3, -1)[:, same], fb.image.view(3, -1)[:, same])
