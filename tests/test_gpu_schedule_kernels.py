"""The frequency map's transforms at the sizes where their branches change, against
the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import schedule as O
from paper_2503_18402_amd import gsmi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,H,W", [
    (1, 1, 1), (1, 1, 2), (2, 3, 5),        # no stage, one stage, an odd row left over
    (1, 61, 122), (1, 67, 134),             # the largest direct prime, the smallest chirp
    (2, 343, 320), (1, 342, 321),           # 64- and 256-thread rows; radices 7, 5, 19
    (1, 64, 1281), (1, 40, 2562),           # 512- and 1024-thread rows
    (1, 1706, 12), (1, 1708, 12),           # three channels of columns at once, one at a time
    (1, 16, 4096), (1, 4093, 7),            # the longest plain and chirp transforms
    (3, 96, 2100),                          # several columns per block
])
def test_transforms_match_oracle(n, H, W):
    imgs = np.random.default_rng(n + H * W).uniform(size=(n, 3, H, W)).astype(np.float32)
    x = torch.from_numpy(imgs).cuda()
    mag = torch.empty(H, W, dtype=torch.float64, device="cuda")
    ws = torch.empty(gsmi.gs_frequency_map_workspace_bytes(H, W), dtype=torch.uint8,
                     device="cuda")
    gsmi.gs_frequency_map(x, H, W, mag, ws)
    ref = np.fft.ifftshift(O.magnitude_map(imgs.astype(np.float64)))
    # each stage of a transform adds a few roundings of a value whose size is the
    # image's 2-norm: 16 roundings for each of up to 2 x 13 stages per axis
    norm = np.sqrt((imgs.astype(np.float64) ** 2).sum(axis=(1, 2, 3))).max()
    assert np.abs(mag.cpu().numpy() - ref).max() <= 16 * 52 * 2.0 ** -53 * norm
