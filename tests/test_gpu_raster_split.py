"""The raster's triangles per wave: launches below, at and above the counts
where one more triangle goes to a wave, and counts that leave the last group of
eight and the last wave incomplete.  The index map is exact."""
import numpy as np
import pytest

from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,L,views", [(1, 1, 1), (3, 3, 1), (511, 4, 1), (512, 4, 1), (513, 4, 1), (911, 3, 2), (1025, 4, 1)])
def test_index_map_over_triangle_counts(P, L, views):
    G.log(f"[raster] P={P} L={L} views={views}")
    sc = S.random_triangles(P=P, degree=2, seed=P)
    cams = S.make_cameras([(0.2, -0.1, 4.0), (2.5, 1.5, 2.8)][:views], [(96, 72), (45, 61)][:views])
    g = G.run_gpu(sc, cams, tile=8, L=L, lean=True)
    po = G.view_offsets(cams)
    for v, fr in enumerate(G.oracle_frames(sc, cams, G.oracle_config(tile=8, L=L))):
        np.testing.assert_array_equal(g["I_tri"][po[v]:po[v + 1]], fr.raster()[0])
