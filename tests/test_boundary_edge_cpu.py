"""The clamp edge of Eq. 7 in FP32: whether a boundary point is in range
(d/sigma < 1) is decided from (d/sigma)^2 by a product with 1/sigma^2, except
within a band around 1, where the quotient itself decides.  Every point that
the two decide differently has to lie in that band."""
import os
import re

import numpy as np

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_13961_amd", "csrc", "bgt_blend.hip")


def test_the_band_holds_every_disagreement():
    src = open(SRC).read()
    band = np.float32(float(re.search(r"kTBand = ([0-9.e+-]+)f", src).group(1)))
    assert re.search(r"kTIn = 1\.0f - 2\.0f \* kTBand, kTOut = 1\.0f \+ 2\.0f \* kTBand", src)
    t_in, t_out = np.float32(1) - np.float32(2) * band, np.float32(1) + np.float32(2) * band
    rng = np.random.default_rng(0)
    f32, n = np.float32, 2_000_000
    sigma = f32(rng.uniform(1.6431677, 60.0, n))  # radii are at least 3 sqrt(0.3)
    ang, q = rng.uniform(0, 2 * np.pi, n), 1.0 + rng.uniform(-3e-7, 3e-7, n)
    dx, dy = f32(q * sigma * np.cos(ang)), f32(q * sigma * np.sin(ang))
    # fma(dx, dx, dy dy) with the product dy dy rounded first
    d2 = f32(dx.astype(np.float64) ** 2 + f32(dy * dy).astype(np.float64))
    t = d2 * (f32(1) / (sigma * sigma))
    quot = np.sqrt(d2) / sigma
    differ = (t < 1) != (quot < 1)
    assert differ.any()  # (so the product alone would decide some of them otherwise)
    assert ((t[differ] >= t_in) & (t[differ] < t_out)).all()
