"""gamma* (Eq. 7) of a boundary list that is longer than the stage: the list is
taken in as many chunks as the tile size asks for (the points within reach of an
8 px tile 88 or 112 at a time, of a 32 px tile 512), and the point whose gamma
counts is the one of smallest d/sigma over the whole list, so the weights, and
with them the images, do not depend on the tile size in any bit.  A planar right
triangle with its legs along a pixel row and column: a pixel on the diagonal
is as far from a point of the row as from one of the column, which lie in
different chunks, up to the rounding of the control points.  The seeds are those
where the smaller d/sigma and the smaller gamma are different points in FP32."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noise,seed", [(1e-6, 30), (3e-6, 3), (1e-5, 53), (1e-5, 5), (3e-5, 44), (3e-5, 29)])
def test_images_do_not_depend_on_the_tile(noise, seed):
    rng = np.random.default_rng(seed)
    W, f, z = 112, 40000.0, 800.0
    cam = H.axis_camera(W, W, f)
    net = np.array([H.pixel_ray_point(cam, x, y, z) for x, y in ((4.2, 4.2), (108.0, 4.2), (4.2, 108.0))])
    sc = H.flat_patch_scene(net, degree=2, log_scale=-3.8, opacity=0.6, sharpness=1e-2 * f / z / rng.uniform(10.0, 12.0))
    sc.ctrl[:] += rng.normal(0.0, noise, sc.ctrl.shape).astype(np.float32)
    sc.color_ctrl[:] = rng.random(sc.color_ctrl.shape, np.float32)
    cams = S.Cameras(cam[None], np.array([[W, W]], np.int32))
    points = {t: int(np.diff(oracle.Frame(sc, cam, W, W, G.oracle_config(tile=t)).lists(1)[0]).max()) for t in (8, 32)}
    G.log(f"[chunks] noise {noise}, seed {seed}: up to {points} points in a tile")
    assert points[8] > 112 and points[32] <= 512
    g = {}
    for tile, batch in ((32, 64), (16, 64), (8, 64), (8, 32)):
        g[tile, batch] = G.run_gpu(sc, cams, tile=tile, batch=batch, pair_factor=64.0, bpair_factor=64.0)
        assert g[tile, batch]["status"] == 0, g[tile, batch]["counters"]
        np.testing.assert_array_equal(g[tile, batch]["images"], g[32, 64]["images"], err_msg=f"tile {tile} batch {batch}")
