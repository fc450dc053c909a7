"""Wide Gaussians of other patches, which a block leaves out of its batches where
none of its pixels shows their patch and no boundary point of theirs is near:
patches that share a bit of the block's set (ids 32 apart), a set of more than
32 patches, a block of background, and the variant without coefficients, where
nothing may be left out.  Images and gradients against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("P,flags", [(2, 0), (33, 0), (65, 0), (150, 0), (65, 1)])
def test_wide_gaussians_of_other_patches(tile, P, flags):
    G.log(f"[own] tile={tile} P={P} flags={flags}")
    sc = S.random_triangles(P=P, degree=2, seed=P + 1)
    sc.log_scale[:] += np.float32(1.8)
    cams = S.make_cameras([(0.2, -0.1, 3.0)], [(75, 61)])
    img_ref, frames = oracle.render_views(sc, cams, G.oracle_config(tile=tile, no_boundary=bool(flags)))
    gi = G.l1_cotangent(img_ref, S.l1_target(cams.num_pixels))
    g = G.run_gpu(sc, cams, tile=tile, flags=flags, grad_images=gi, pair_factor=64.0, bpair_factor=64.0)
    assert g["status"] == 0, g["counters"]
    assert np.abs(g["images"] - img_ref).max() <= 1e-4
    G.check_grads(g["grads"], oracle.grad_views(frames, gi))
