"""The frequency map's transforms and the strip downsampling at the sizes where
their branches change, against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import schedule as O
from paper_2503_18402_amd import gsmi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,H,W", [
    (1, 1, 1), (1, 1, 2), (2, 3, 5),        # no stage, one stage, an odd row left over
    (1, 61, 122), (1, 134, 134),            # the largest direct prime, the smallest chirp
    (1, 67, 134),
    (2, 40, 104), (2, 41, 104),             # the last sums without transforms, the first with
    (1, 67, 189), (1, 67, 190), (1, 150, 67),   # the same where a line would need a chirp
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


@pytest.mark.parametrize("H,W,h,w", [
    (64, 64, 64, 64), (65, 67, 65, 33),     # factor 1 on both axes, on one
    (90, 120, 30, 40), (91, 121, 30, 40),   # rows 16-byte aligned or not
    (33, 4100, 11, 2050), (12, 4096, 5, 20),   # several column tiles; a wide window
    (2000, 8, 16, 8), (1260, 12, 10, 5), (1270, 12, 10, 5),  # 1 row per strip, the last strip
                                            # factor, and one thread per output past it
    (17, 3000, 17, 2), (9, 9, 1, 1), (5, 7, 8, 3),
    (5600, 16, 2800, 8), (5600, 20, 2733, 5), (5601, 17, 2800, 8),   # 16 rows per strip
    (400, 16, 200, 8), (1600, 20, 800, 10), (2800, 17, 1400, 8),     # 2, 4 and 8 rows
    (60, 128, 48, 100), (60, 130, 30, 65), (64, 512, 8, 64),  # one and several columns a
                                            # thread, its four in one LDS plane or in four
])
def test_downsample_strips_match_oracle(H, W, h, w):
    x = np.random.default_rng(H * w).uniform(size=(2, 3, H, W)).astype(np.float32)
    src = torch.from_numpy(x).cuda()
    dst = torch.full((6 * h * w,), -1.0, device="cuda")
    gsmi.gs_downsample_aa(src, 6, H, W, h, w, dst)
    got = dst.view(2, 3, h, w).cpu().numpy()
    ref = np.stack([O.downsample_aa(x[k].astype(np.float64), h, w) for k in range(2)])
    # FP64 sums of values in [0, 1): one float32 rounding
    assert np.abs(got - ref).max() <= 2.0 ** -24


def test_downsample_rows_of_weight_zero_are_not_read():
    """At an odd integer factor a row can sit exactly one window from a centre:
    its infinities stay out of that output row."""
    x = torch.rand(1, 3, 30, 32, device="cuda")
    x[:, :, 4] = float("inf")     # the centre of output row 1: weight 0 in rows 0 and 2
    dst = torch.empty(3 * 10 * 32, device="cuda")
    gsmi.gs_downsample_aa(x, 3, 30, 32, 10, 32, dst)
    row = dst.view(3, 10, 32).isfinite().all(2).all(0).cpu().numpy()
    assert (row == (np.arange(10) != 1)).all()
