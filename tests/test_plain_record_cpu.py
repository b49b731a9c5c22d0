"""The blend kernels' rule for plain records, in float32 on the CPU: a record that it
accepts has an exponent p2 <= 0 at every pixel offset, also where the conic is nearly
singular and the offset runs along its long axis, and an alpha below the clamp."""
import re
from pathlib import Path

import numpy as np

F = np.float32
CSRC = Path(__file__).resolve().parents[1] / "paper_2503_18402_amd" / "csrc"


def _fma(a, b, c):  # the product is exact in float64
    return (a.astype(np.float64) * b.astype(np.float64) + c).astype(F)


def test_plain_records_never_need_the_general_walk():
    src = (CSRC / "blend_common.hpp").read_text()
    assert "(d - r0.w * r0.w > 1.0e-4f * d)" in src and "kLog2AlphaMax - 1.0e-4f" in src
    log2_max = float(re.search(r"kLog2AlphaMax = (-[0-9.]+)f", (CSRC / "gs_internal.hpp")
                               .read_text()).group(1))
    assert 2.0 ** (log2_max - 1.0e-4) * (1 + 2.0 ** -20) < 0.99
    rng = np.random.default_rng(0)
    n = 1 << 20
    for rep in range(4):
        a, c = 10.0 ** rng.uniform(-6, 1, n), 10.0 ** rng.uniform(-6, 1, n)
        rho = np.sqrt(1.0 - 10.0 ** rng.uniform(-7, 0, n)) * rng.choice([-1, 1], n)
        A, C, B = F(-a), F(-c), F(-2 * rho * np.sqrt(a * c))
        d = F(4) * A * C
        plain = (A < 0) & (C < 0) & (d - B * B > F(1e-4) * d)
        assert 0.3 < plain.mean() < 0.9
        # along the long axis (p2 closest to 0) and slightly off it
        t = 10.0 ** rng.uniform(-2, 4, n) * rng.choice([-1, 1], n)
        dx = F(t * np.sqrt(c / a)) if rep % 2 else F(t)
        dy = F(-dx * np.sign(rho) * np.sqrt(a / c) * (1 + rng.normal(0, 1e-3, n) * (rep > 1)))
        t1 = _fma(A, dx, (B * dy))
        p2 = _fma(dx, t1, (C * dy) * dy)
        assert (p2[plain] <= 0).all()
    assert (p2 > 0).any()  # the offsets do reach the rounding that the rule is for
