"""The oracle's Eq. 5 interpolation just past the patch's rim: a pixel that the
snapped edge covers can lie past u + v = 1 by the snap, where the map has no
further texel.  The three texels stay those of the hypotenuse cell, and a linear
map is reproduced there as inside."""
import numpy as np
import pytest


@pytest.mark.parametrize("u,v", [(0.5003, 0.5001), (0.75, 0.2505), (0.9999, 0.0003), (0.25, 0.7504), (0.0004, 0.9999),
                                 (0.4999, 0.5004)])
def test_theta_past_the_rim(orc, u, v):
    nodes = np.array([(a / 2, b / 2) for a in range(3) for b in range(3 - a)])  # lattice order, a outer
    ti, tw = orc.theta(3, u, v)
    assert set(ti) <= set(range(6)), ti
    assert abs(tw.sum() - 1.0) < 1e-15
    np.testing.assert_allclose(tw @ nodes[ti], (u, v), atol=1e-15)
