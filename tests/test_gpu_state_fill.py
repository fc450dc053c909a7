"""The state buffer's former content may not show in a pass: forward and backward
from a buffer of NaN and from one of zeros.  Attribute maps where pixels of the
last patch lie just past u + v = 1 (its edge, snapped to 1/256 px, reaches a column
of pixel centres) read the words after the patch records; a lattice and a scene with
lists beyond the stage take every other section.  Images in every bit, gradients
up to the order of float atomics."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _rim(degree, P):
    W, Hh = 32, 24
    cam = H.axis_camera(W, Hh, 32.0)
    # corners of u = 1, v = 1, w = 1 (pixel, depth; tilted, so that the Gaussians' depths differ): the
    # edge u + v = 1 is 0.001 px short of the centres of column 20
    net = np.array([H.pixel_ray_point(cam, *p) for p in ((20.499, 2.3, 2.0), (20.499, 21.7, 2.1), (14.2, 12.1, 2.35))])
    one = H.flat_patch_scene(net, degree=degree, log_scale=-2.5)
    off = H.flat_patch_scene(net - np.array([0.0, 0.0, 10.0]), degree=degree)  # behind the camera
    sc = S.with_attributes(S.concat([off] * (P - 1) + [one]), attr_res=3, sh_degree=0, seed=4)
    it, uv, _, _ = oracle.Frame(sc, cam, W, Hh, G.oracle_config(tile=8)).raster()
    rim = (it >= 0) & (uv.sum(1) > 1.0 + 1e-5)
    assert (it[rim] // 16 == P - 1).all() and ((2.0 * uv[rim, 0]) >= 1.0).sum() >= 8
    return sc, S.Cameras(cam[None], np.array([[W, Hh]], np.int32)), {}


def _dense(**config):
    sc = S.random_triangles(P=300, degree=2, seed=5)
    sc.sharpness[:] = 0.5
    return sc, S.make_cameras([(0.2, -0.1, 2.5)], [(72, 56)]), config


@pytest.mark.parametrize("make", [lambda: _rim(1, 2), lambda: _rim(2, 4), lambda: _rim(3, 2), lambda: _dense(tile=8),
                                  lambda: _dense(tile=16), lambda: _dense(tile=16, lattice=3)])
def test_pass_does_not_depend_on_the_buffer(make):
    import torch
    from paper_2503_13961_amd.render import Renderer, scene_tensors
    sc, cams, config = make()
    G.log(f"[fill] degree {sc.degree}, {sc.num_prims} patches, {config}")
    dev = torch.device("cuda", 0)
    r = Renderer(0, **({"tile": 8} | config), pair_factor=64.0, bpair_factor=64.0)
    params, camt = scene_tensors(sc, dev), torch.from_numpy(cams.cams).to(dev)
    gi = torch.from_numpy(S.l1_target(cams.num_pixels).astype(np.float32)).to(dev) - 0.5
    out = []
    for fill in (0, 0xFF):
        state = torch.full((r.state_bytes(sc.degree, params, camt, cams.wh),), fill, dtype=torch.uint8, device=dev)
        img, _ = r.forward(sc.degree, params, camt, cams.wh, state=state)
        grads = r.backward(sc.degree, params, camt, cams.wh, img, gi, state)
        out.append((img.cpu().numpy(), {k: v.cpu().numpy() for k, v in grads.items()}))
    (a, ga), (b, gb) = out
    assert np.isfinite(a).all()
    np.testing.assert_array_equal(a, b)
    for k in ga:
        assert np.isfinite(ga[k]).all() and G.grad_error(gb[k], ga[k]) <= 1e-5, k
