"""The splitting statistics of large launches, which sum over regions of 32 px
(from 1024 of them on; smaller launches over regions of 16 px): one view and
ragged views whose sizes leave the last regions incomplete, with and without
targets, and for both sizes of region one that shows more patches than its table
takes, so that the rest is added to memory.  Tolerances as for the other
statistics tests: counts and bits exact, the sums of FP32 magnitudes within 1e-5
of the largest."""
import numpy as np
import pytest

from oracle import densify as D
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

ROWS, PROBES = 256, 16


def table_misses(prims, order):
    """Patches that find no row in the region's table, added in this order."""
    table, misses = {}, 0
    for p in prims[order]:
        h = ((int(p) * 2654435761) & 0xFFFFFFFF) >> 16
        for n in range(PROBES):
            if table.setdefault((h + n) % ROWS, p) == p:
                break
        else:
            misses += 1
    return misses


@pytest.mark.parametrize("wh,side,freq,L,dist", [
    ([(1100, 1000)], 32, 40, 2, 10.0),             # 1120 regions, many with a full table
    ([(1500, 700), (333, 77)], 32, 10, 4, 2.2),   # 1067 regions
    ([(200, 180)], 16, 40, 2, 6.0),               # 13x12 regions of 16 px, full tables
])
def test_statistics_of_large_launches(wh, side, freq, L, dist):
    import torch
    from paper_2503_13961_amd.densify import PrimStats
    from paper_2503_13961_amd.render import Renderer, scene_tensors
    assert (sum(-(-w // 32) * -(-h // 32) for w, h in wh) >= 1024) == (side == 32)
    sc = S.deformed_sphere(freq=freq, degree=2, seed=3, noise=0.02)
    cams = S.make_cameras([(0.3 * dist, -0.2 * dist, 0.93 * dist), (-0.8 * dist, 0.1 * dist, 0.6 * dist)][:len(wh)], wh)
    its = [fr.raster()[0] for fr in G.oracle_frames(sc, cams, G.oracle_config(tile=8, L=L))]
    if freq == 40:
        it = its[0].reshape(wh[0][1], wh[0][0]) // (L * L)
        y, x = (side * int(d // side // 2) for d in it.shape)  # a region in the middle of the sphere
        prims = np.unique(it[y:y + side, x:x + side])
        assert prims[0] >= 0
        rng = np.random.default_rng(0)
        misses = [table_misses(prims, rng.permutation(len(prims))) for _ in range(8)]
        G.log(f"[stats] {len(prims)} patches in the {side} px region at ({x}, {y}): {min(misses)} to {max(misses)} without a row")
        assert min(misses) > 0
    dev = torch.device("cuda", 0)
    r = Renderer(0, tile=8, tess_level=L)
    params, camt = scene_tensors(sc, dev), torch.from_numpy(cams.cams).to(dev)
    _, state = r.forward(sc.degree, params, camt, cams.wh)
    targets = np.random.default_rng(2).random((cams.num_pixels, 3)).astype(np.float32)
    ref = D.Stats(sc.num_prims, L)
    ref.accumulate(its, [tuple(int(x) for x in w) for w in cams.wh], targets)
    for with_targets in (True, False):
        st = PrimStats(sc.num_prims, dev)
        st.accumulate(r, sc.degree, params, camt, cams.wh, state, torch.from_numpy(targets).to(dev) if with_targets else None)
        got = {k: v.cpu().numpy() for k, v in st.t.items()}
        np.testing.assert_array_equal(got["vis_views"], ref.vis_views)
        np.testing.assert_array_equal(got["tex"].view(np.uint64), ref.tex)
        if with_targets:
            np.testing.assert_array_equal(got["edge_cnt"], ref.edge_cnt)
            assert np.abs(got["edge_sum"] - ref.edge_sum).max() <= 1e-5 * np.abs(ref.edge_sum).max()
        else:
            assert not got["edge_cnt"].any() and not got["edge_sum"].any()
