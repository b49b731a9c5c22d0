"""The chain rule's gradient slabs at their edges: fewer Gaussians than a block, one more
than one, a last block of one; every SH degree, whose 3, 12, 27 or 48 values end inside a
16-byte piece or at one; written over and added to; SH gradients at a 4-byte offset.
The same kernel writes both forms, so they agree bit for bit: g written over NaN, and
x + g added to x, with x untouched above the degree and where no pair reaches."""
import pytest
import torch

from paper_2503_18402_amd import gsmi, raster, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 127, 129, 1000])
@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("shift", [0, 1])
def test_written_and_added_gradients_agree(n, degree, shift):
    sc = scenes.make_scene(n, seed=n, mean_range=0.6, ls_mu=-2.5)
    sc["means"][n // 2:n // 2 + 3] += 90.0  # out of view
    cam = scenes.look_at((0, 0, -3.0), (0, 0, 0), 80, 56, 70.0)
    params = raster.to_device(sc)
    frame = raster.render(params, [cam], sh_degree=degree)
    dL = torch.from_numpy(scenes.random_upstream(cam, seed=5)).reshape(-1).cuda()
    gen = torch.Generator(device="cuda").manual_seed(3)

    def grads(fill):
        g = {k: fill(v) for k, v in params.items()}
        flat = torch.empty(48 * n + 4, device="cuda")[shift:shift + 48 * n].view(n, 16, 3)
        g["sh"] = flat.copy_(g["sh"])
        return g

    base = raster.render_backward(params, frame, dL)           # added to zeros
    over = raster.render_backward(params, frame, dL, accumulate=False,
                                  grads=grads(lambda v: torch.full_like(v, float("nan"))))
    x = grads(lambda v: torch.randn(v.shape, device="cuda", generator=gen))
    want = {k: x[k] + base[k] for k in x}
    added = raster.render_backward(params, frame, dL, grads=x)
    torch.cuda.synchronize()
    seen = torch.count_nonzero(base["means"].abs().sum(1)).item()
    assert 0 < seen <= n or n <= 3
    K = (degree + 1) ** 2
    assert not over["sh"][:, K:].any()
    for k in raster.PARAM_NAMES:
        assert torch.equal(over[k], base[k]), k
        assert torch.equal(added[k], want[k]), k
