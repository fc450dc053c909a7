"""The blend kernels' rows of boundary weights where a tile has more of them
than LDS holds (memory from the pool), more than the pool holds or more runs than
the run table (searched per pixel), and lists longer than the stage (taken in
chunks): images and gradients against the oracle, with ample pair capacities
and with capacities that just hold the lists (the pool is what they leave)."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,batch", [(8, 32), (8, 64), (16, 64), (32, 64)])
@pytest.mark.parametrize("P,sharpness", [(500, 1.0), (900, 0.1), (900, 0.03)])
def test_rows_beyond_lds(tile, batch, P, sharpness):
    sc = S.random_triangles(P=P, degree=2, seed=P)
    sc.sharpness[:] = np.float32(sharpness)
    cams = S.make_cameras([(0.2, -0.1, 2.5)], [(72, 56)])
    img_ref, frames = oracle.render_views(sc, cams, G.oracle_config(tile=tile))
    (gof, _), (bof, blst) = frames[0].lists(0), frames[0].lists(1)
    prim = frames[0].raster()[0] // 16
    runs = max(len(np.unique(prim[blst[bof[i]:bof[i + 1]]])) for i in range(len(bof) - 1))
    G.log(f"[rows] tile={tile} batch={batch}: up to {runs} runs and {np.diff(bof).max()} points in a tile")
    assert runs > 12
    gi = G.l1_cotangent(img_ref, S.l1_target(cams.num_pixels))
    ref = oracle.grad_views(frames, gi)
    n = cams.num_pixels
    just = {k: max((off[-1] - 1000) / n, 1e-3) for k, off in (("pair_factor", gof), ("bpair_factor", bof))}
    for caps in (dict(pair_factor=64.0, bpair_factor=64.0), just):
        g = G.run_gpu(sc, cams, tile=tile, batch=batch, grad_images=gi, **caps)
        assert g["status"] == 0, g["counters"]
        assert np.abs(g["images"] - img_ref).max() <= 1e-4
        G.check_grads(g["grads"], ref)
