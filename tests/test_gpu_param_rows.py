"""The parameter pass where a 32x32 region shows more patches than its table
has rows (their sums then go to the patch's words one by one), with patches of
every pixel count per 8x8 block, and patch counts that leave the last 64 of the
gradient transpose incomplete.  Gradient measures as for the other parity tests."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,degree,res,sh", [(901, 2, 1, 0), (900, 1, 1, 0), (831, 3, 1, 0), (700, 2, 3, 3), (577, 5, 1, 2)])
def test_more_patches_than_table_rows(P, degree, res, sh):
    G.log(f"[param] P={P} degree={degree} R={res} SH={sh}")
    sc = S.random_triangles(P=P, degree=degree, seed=P)
    if res > 1 or sh > 0:
        sc = S.with_attributes(sc, attr_res=res, sh_degree=sh, seed=P, sh_std=0.2)
    cams = S.make_cameras([(0.2, -0.1, 2.5), (2.5, 1.5, 2.8)], [(64, 64), (33, 47)])
    img_ref, frames = oracle.render_views(sc, cams, G.oracle_config(tile=8))
    it = frames[0].raster()[0].reshape(64, 64)
    seen = max(len(np.unique(b[b >= 0] // 16)) for b in (it[j:j + 32, i:i + 32] for j in (0, 32) for i in (0, 32)))
    G.log(f"    up to {seen} patches in a 32x32 region")
    assert seen > 64
    gi = G.l1_cotangent(img_ref, S.l1_target(cams.num_pixels))
    g = G.run_gpu(sc, cams, tile=8, grad_images=gi)
    G.check_grads(g["grads"], oracle.grad_views(frames, gi))
