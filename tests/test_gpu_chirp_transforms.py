"""The frequency map where a line has a large prime factor and goes through a chirp
convolution, against numpy's transforms in long double: no further off than the direct sums
are, whose error on such images is 2 to 3.5e-16 of the map's 2-norm and less over several;
and at the lengths whose convolutions take other stages, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import schedule as O
from paper_2503_18402_amd import gsmi

pytestmark = pytest.mark.gpu


def _map(imgs):
    n, _, H, W = imgs.shape
    mag = torch.empty(H, W, dtype=torch.float64, device="cuda")
    ws = torch.empty(gsmi.gs_frequency_map_workspace_bytes(H, W), dtype=torch.uint8, device="cuda")
    gsmi.gs_frequency_map(torch.from_numpy(imgs).cuda(), H, W, mag, ws)
    return mag.cpu().numpy()


@pytest.mark.parametrize("n,H,W", [(1, 211, 263), (1, 134, 402), (2, 401, 503), (1, 607, 809),
                                   (4, 607, 809), (1, 4093, 300)])
def test_error_is_that_of_direct_sums(n, H, W):
    g = torch.Generator().manual_seed(H * W)
    low = torch.rand(n, 3, H // 16 + 2, W // 16 + 2, generator=g)
    img = torch.nn.functional.interpolate(low, (H, W), mode="bilinear", align_corners=True)
    imgs = (0.9 * img + 0.1 * torch.rand(n, 3, H, W, generator=g)).numpy()
    got = _map(imgs)
    F = np.fft.fft2(imgs.astype(np.longdouble), axes=(2, 3))
    assert F.dtype == np.clongdouble
    ref = np.sqrt((F.real ** 2 + F.imag ** 2).sum(1)).mean(0)
    err = np.sqrt(((got - ref) ** 2).sum() / (ref ** 2).sum())
    assert err <= 2.0 ** -52, float(err)


@pytest.mark.parametrize("n,H,W", [(1, 67, 331), (2, 211, 167), (1, 199, 263), (1, 1009, 71),
                                   (1, 2503, 16), (2, 16, 4093)])
def test_chirps_match_oracle(n, H, W):
    imgs = np.random.default_rng(H + W).uniform(size=(n, 3, H, W)).astype(np.float32)
    ref = np.fft.ifftshift(O.magnitude_map(imgs.astype(np.float64)))
    norm = np.sqrt((imgs.astype(np.float64) ** 2).sum(axis=(1, 2, 3))).max()
    # 16 roundings of the 2-norm for each of up to 2 x 13 stages per axis
    assert np.abs(_map(imgs) - ref).max() <= 16 * 52 * 2.0 ** -53 * norm


@pytest.mark.parametrize("n,H,W,kernel", [(1, 71, 211, "k_dft_rows"), (2, 131, 189, "k_dft_rows"),
                                          (2, 131, 190, "k_fft_rows")])
def test_small_views_are_summed(n, H, W, kernel):
    """Up to 320 values of both lines together the sums take no longer than the chirps,
    for one view and for several."""
    imgs = np.random.default_rng(H + W).uniform(size=(n, 3, H, W)).astype(np.float32)
    torch.cuda.synchronize()
    gsmi.gs_profile_enable(True)
    got = _map(imgs)
    times = gsmi.gs_profile_collect()
    gsmi.gs_profile_enable(False)
    assert kernel in times, times
    ref = np.fft.ifftshift(O.magnitude_map(imgs.astype(np.float64)))
    norm = np.sqrt((imgs.astype(np.float64) ** 2).sum(axis=(1, 2, 3))).max()
    assert np.abs(got - ref).max() <= 16 * 52 * 2.0 ** -53 * norm


@pytest.mark.parametrize("n,H,W,sums", [(4, 61, 122, True), (1, 59, 118, True), (1, 37, 111, False),
                                        (1, 799, 16, False), (1, 901, 16, False)])
def test_large_stages_match_oracle(n, H, W, sums):
    """Primes of 41 to 61 have a stage of their own in lines of more than 800 values only:
    a small view of such lines is summed (four of 61x122 took 102 us through them, 80 before
    there were transforms, 50 so)."""
    imgs = np.random.default_rng(H + W).uniform(size=(n, 3, H, W)).astype(np.float32)
    torch.cuda.synchronize()
    gsmi.gs_profile_enable(True)
    got = _map(imgs)
    times = gsmi.gs_profile_collect()
    gsmi.gs_profile_enable(False)
    assert ("k_dft_rows" in times) == sums, times
    ref = np.fft.ifftshift(O.magnitude_map(imgs.astype(np.float64)))
    norm = np.sqrt((imgs.astype(np.float64) ** 2).sum(axis=(1, 2, 3))).max()
    assert np.abs(got - ref).max() <= 16 * 52 * 2.0 ** -53 * norm
