"""Forward and backward where the waves of a tile go through its list at
different paces: lists of a few to several hundred entries (less than one batch
to several rounds of the backward's ring of batches), pixels that replay
nothing (no cotangent on some 8x8 blocks, none on whole tiles), records that
reach more than 3x3 tiles, views that leave blocks of a tile outside."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("widen", [0.0, 1.2, 2.6])
def test_waves_at_their_own_pace(tile, widen):
    G.log(f"[blend] tile={tile} widen={widen}")
    sc = S.random_triangles(P=48, degree=2, seed=21)
    sc.log_scale[:] += np.float32(widen)
    cams = S.make_cameras([(0.2, -0.1, 3.0), (2.5, 1.5, 2.8)], [(97, 70), (41, 23)])
    img_ref, frames = oracle.render_views(sc, cams, G.oracle_config(tile=tile))
    gi = G.l1_cotangent(img_ref, S.l1_target(cams.num_pixels))
    v0 = gi[:97 * 70].reshape(70, 97, 3)
    v0[8:16, 24:48] = 0.0   # blocks of a tile without a cotangent
    v0[32:64, 32:64] = 0.0  # a whole tile of 32
    v0[:, 8:16] = 0.0
    g = G.run_gpu(sc, cams, tile=tile, grad_images=gi)
    assert g["status"] == 0, g["counters"]
    G.log(f"    lists of up to {g['g_count'].max()} entries")
    assert np.abs(g["images"] - img_ref).max() <= 1e-4
    G.check_grads(g["grads"], oracle.grad_views(frames, gi))
