"""The launch before the raster (clears, patch records, projected lattice) and
the scan of the tile counts at the sizes where they change their split: a
lattice point shared by four views with a remainder, tile counts at the edges
of a scan round, of the one-launch scan and of the tile order, few patches."""
import numpy as np
import pytest

from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def test_lattice_points_shared_by_views():
    P, L, n = 18700, 8, 5
    assert P * (L + 1) * (L + 2) // 2 * n >= 1 << 22
    G.log(f"[front] {P} patches, {n} views")
    sc = S.random_triangles(P=P, degree=2, seed=2)
    cams = S.make_cameras(S.fibonacci_eyes(n, 4.0), [(40, 30), (33, 21), (8, 8), (1, 17), (37, 29)])
    g = G.run_gpu(sc, cams, tile=8, L=L, lean=True)
    po = G.view_offsets(cams)
    for v, fr in enumerate(G.oracle_frames(sc, cams, G.oracle_config(tile=8, L=L))):
        np.testing.assert_array_equal(g["I_tri"][po[v]:po[v + 1]], fr.raster()[0])


@pytest.mark.parametrize("wh", [[(504, 520)], [(512, 512)], [(512, 512), (5, 3)], [(1024, 1024)], [(1024, 1024), (5, 3)],
                                [(1, 1)], [(256, 256)], [(264, 256)]])
def test_segments_over_tile_counts(wh):
    G.log(f"[scan] views {wh}")
    sc = S.random_triangles(P=16, degree=2, seed=5)
    cams = S.make_cameras([(0.2, -0.1, 4.0), (2.5, 1.5, 2.8)][:len(wh)], wh)
    g = G.run_gpu(sc, cams, tile=8)
    assert g["status"] == 0, g["counters"]
    to, po = G.tile_offsets(cams, 8), G.view_offsets(cams)
    for v, fr in enumerate(G.oracle_frames(sc, cams, G.oracle_config(tile=8))):
        for which, n in enumerate("gb"):
            np.testing.assert_array_equal(g[n + "_count"][to[v]:to[v + 1]], np.diff(fr.lists(which)[0]))
        # (every tile has a place in the blend's order)
        assert np.abs(g["images"][po[v]:po[v + 1]] - fr.render()[0]).max() <= 1e-4
    for i, n in enumerate("gb"):
        total = np.cumsum(g[n + "_count"].astype(np.int64))
        np.testing.assert_array_equal(g[n + "_start"], total - g[n + "_count"])
        assert g["counters"][1 + i] == total[-1]
