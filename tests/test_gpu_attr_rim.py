"""Attribute maps where pixels of the last patch lie just past u + v = 1 (its
edge, snapped to 1/256 px, reaches a column of pixel centres): the maps end with
the texels of that patch, so nothing that the state buffer held before may show
in the image or the gradients.  Against the oracle, from a buffer of NaN and
from one of zeros; tolerances as for the other parity tests."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree,P", [(1, 2), (2, 4), (3, 2)])
def test_rim_pixels_of_the_last_patch(degree, P):
    import torch
    from paper_2503_13961_amd.render import Renderer, scene_tensors
    G.log(f"[attr] rim, degree {degree}")
    W, Hh = 32, 24
    cam = H.axis_camera(W, Hh, 32.0)
    # corners of u = 1, v = 1, w = 1 (pixel, depth; tilted, so that the Gaussians' depths differ): the
    # edge u + v = 1 is 0.001 px short of the centres of column 20
    net = np.array([H.pixel_ray_point(cam, *p) for p in ((20.499, 2.3, 2.0), (20.499, 21.7, 2.1), (14.2, 12.1, 2.35))])
    one = H.flat_patch_scene(net, degree=degree, log_scale=-2.5)
    off = H.flat_patch_scene(net - np.array([0.0, 0.0, 10.0]), degree=degree)  # behind the camera
    sc = S.concat([off] * (P - 1) + [one])
    sc = S.with_attributes(sc, attr_res=3, sh_degree=0, seed=4)
    cams = S.Cameras(cam[None], np.array([[W, Hh]], np.int32))
    img_ref, frames = oracle.render_views(sc, cams, G.oracle_config(tile=8))
    it, uv, _, _ = frames[0].raster()
    rim = (it >= 0) & (uv.sum(1) > 1.0 + 1e-5)
    assert (it[rim] // 16 == P - 1).all() and rim.sum() >= 8, rim.sum()
    assert (2.0 * uv[rim, 0] >= 1.0).any() and (2.0 * uv[rim, 0] < 1.0).any()  # both hypotenuse cells
    gi = G.l1_cotangent(img_ref, S.l1_target(cams.num_pixels))
    ref = oracle.grad_views(frames, gi)
    dev = torch.device("cuda", 0)
    r = Renderer(0, tile=8)
    params, camt = scene_tensors(sc, dev), torch.from_numpy(cams.cams).to(dev)
    nbytes = r.state_bytes(degree, params, camt, cams.wh)
    for fill in (0xFF, 0):
        state = torch.full((nbytes,), fill, dtype=torch.uint8, device=dev)
        img, _ = r.forward(degree, params, camt, cams.wh, state=state)
        grads = r.backward(degree, params, camt, cams.wh, img, torch.from_numpy(gi.astype(np.float32)).to(dev), state)
        assert np.abs(img.cpu().numpy() - img_ref).max() <= 1e-4
        G.check_grads({k: v.cpu().numpy() for k, v in grads.items()}, ref)
