"""The raster's triangles per wave in larger launches: counts just below, at and
above those where a wave takes 8, 16, 32 and 64 (from 8 on it takes whole groups of
the launch's permutation).  The index map is exact."""
import numpy as np
import pytest

from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [n + d for n in (512, 1024, 2048, 4096) for d in (-1, 0, 1)])
def test_index_map_over_larger_triangle_counts(P):
    G.log(f"[raster] P={P}: {64 * P} triangles")
    assert 64 * 512 == 8 * 4096  # (4096 waves of 8)
    sc = S.random_triangles(P=P, degree=1, seed=P)
    cams = S.make_cameras([(0.2, -0.1, 4.0)], [(61, 53)])
    g = G.run_gpu(sc, cams, tile=8, L=8, lean=True)
    fr, = G.oracle_frames(sc, cams, G.oracle_config(tile=8, L=8))
    np.testing.assert_array_equal(g["I_tri"], fr.raster()[0])
