"""Tile lists at the lengths where the sort changes its method: one workgroup's
buffer (2048), several buffers ranked against each other with a last one of
any length (a few keys, one run of 512, more), and more buffers than are
ranked.  Every boundary point reaches every tile, so that a list is as long as
the view has boundary points; the order is bit-exact against the oracle's."""
import numpy as np
import pytest

from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,wh,lo,hi", [(64, (50, 41), 512, 1024), (64, (80, 70), 1024, 2048), (64, (128, 96), 2048, 2560),
                                        (64, (200, 190), 4096, 6144), (1500, (330, 320), 14 * 2048, 16 * 2048),
                                        (4000, (470, 460), 65536, 1 << 20)])
def test_list_lengths(P, wh, lo, hi):
    sc = S.random_triangles(P=P, degree=2, seed=1)
    sc.sharpness[:] = np.float32(0.002)
    cams = S.make_cameras([(0.0, 0.0, 2.5)], [wh])
    fr = G.oracle_frames(sc, cams, G.oracle_config(tile=32))[0]
    off, lst = fr.lists(1)
    n = int(np.diff(off).max())
    G.log(f"[sort] {n} boundary points in every tile's list")
    assert lo < n <= hi
    g = G.run_gpu(sc, cams, tile=32, bpair_factor=float(len(off)))
    assert g["status"] == 0, g["counters"]
    np.testing.assert_array_equal(g["b_count"], np.diff(off))
    np.testing.assert_array_equal(g["b_list"], lst)
    off, lst = fr.lists(0)
    np.testing.assert_array_equal(g["g_count"], np.diff(off))
    np.testing.assert_array_equal(g["g_list"], lst)
