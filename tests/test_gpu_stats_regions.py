"""The splitting statistics where a 32x32 region shows more patches than its
table has rows, at 64 sub-triangles per patch (both words of the visibility
texture), and on views that leave regions incomplete or are smaller than one.
Tolerances as for the other statistics tests: counts and bits exact, the sums
of FP32 magnitudes within 1e-5 of the largest."""
import numpy as np
import pytest

from oracle import densify as D
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,wh", [(8, [(64, 64), (33, 47)]), (4, [(5, 3), (65, 31)]), (5, [(1, 40), (96, 1)])])
def test_statistics_over_regions(L, wh):
    import torch
    from paper_2503_13961_amd.densify import PrimStats
    from paper_2503_13961_amd.render import Renderer, scene_tensors
    G.log(f"[densify] regions, L={L}, views {wh}")
    sc = S.random_triangles(P=900, degree=2, seed=901)
    cams = S.make_cameras([(0.2, -0.1, 2.5), (2.5, 1.5, 2.8)], wh)
    dev = torch.device("cuda", 0)
    r = Renderer(0, tile=8, tess_level=L)
    params, camt = scene_tensors(sc, dev), torch.from_numpy(cams.cams).to(dev)
    _, state = r.forward(sc.degree, params, camt, cams.wh)
    targets = np.random.default_rng(2).random((cams.num_pixels, 3)).astype(np.float32)
    st = PrimStats(sc.num_prims, dev)
    st.accumulate(r, sc.degree, params, camt, cams.wh, state, torch.from_numpy(targets).to(dev))
    got = {k: v.cpu().numpy() for k, v in st.t.items()}
    its = [fr.raster()[0] for fr in G.oracle_frames(sc, cams, G.oracle_config(tile=8, L=L))]
    if wh[0] == (64, 64):
        b = its[0].reshape(64, 64)[:32, :32]
        assert len(np.unique(b[b >= 0] // (L * L))) > 64
    ref = D.Stats(sc.num_prims, L)
    ref.accumulate(its, [tuple(int(x) for x in w) for w in cams.wh], targets)
    np.testing.assert_array_equal(got["vis_views"], ref.vis_views)
    np.testing.assert_array_equal(got["tex"].view(np.uint64), ref.tex)
    np.testing.assert_array_equal(got["edge_cnt"], ref.edge_cnt)
    assert np.abs(got["edge_sum"] - ref.edge_sum).max() <= 1e-5 * max(np.abs(ref.edge_sum).max(), 1e-30)
