"""The generation's two ways of reading patch records (one or two patches in an
8x8 block: scalar loads; more: per lane) and the pair counts within and beyond
the 3x3 tiles around a block, at the image's borders: bit-exact index map and
tile lists, images within 1e-4."""
import numpy as np
import pytest

from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("P,degree,widen", [(1, 1, 0.0), (2, 2, 1.5), (3, 4, 0.0), (40, 2, 1.5), (300, 3, 0.0)])
def test_lists_over_patches_per_block(P, degree, widen, tile):
    G.log(f"[gen] P={P} degree={degree} widen={widen} tile={tile}")
    sc = S.random_triangles(P=P, degree=degree, seed=3 + P)
    sc.log_scale[:] += np.float32(widen)  # (Gaussians of a few tiles of 8)
    cams = S.make_cameras([(0.2, -0.1, 2.5), (2.5, 1.5, 2.8)], [(65, 50), (23, 40)])
    g = G.run_gpu(sc, cams, tile=tile)
    assert g["status"] == 0, g["counters"]
    po, to = G.view_offsets(cams), G.tile_offsets(cams, tile)
    for v, fr in enumerate(G.oracle_frames(sc, cams, G.oracle_config(tile=tile))):
        it, iu, _, val = fr.raster()
        sl = slice(po[v], po[v + 1])
        np.testing.assert_array_equal(g["I_tri"][sl], it)
        assert np.abs(g["I_uv"][sl][it >= 0] - iu[it >= 0]).max(initial=0) < 1e-6
        for which, n in enumerate("gb"):
            off, lst = fr.lists(which)
            cnt, start = g[n + "_count"][to[v]:to[v + 1]], g[n + "_start"][to[v]:to[v + 1]]
            np.testing.assert_array_equal(cnt, np.diff(off))
            for t in range(len(cnt)):
                np.testing.assert_array_equal(g[n + "_list"][start[t]:start[t] + cnt[t]] - po[v], lst[off[t]:off[t + 1]])
        assert np.abs(g["images"][sl] - fr.render()[0]).max() <= 1e-4
