"""bgt_query's count of tiles with more boundary runs than the forward keeps
weights of in LDS: 8 px tiles by their runs, larger ones by the runs that reach
one of their 8x8 blocks, as the rows are kept.  Against the same rule over the
oracle's lists (a point reaches the pixels of its radius and one more each side)."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def expected(fr, tile, rows, widen=0.0):
    """(tiles counted, tiles with more than `rows` runs) of the tiles with Gaussians."""
    rec, (gof, _), (bof, blst) = fr.records(), fr.lists(0), fr.lists(1)
    counted = many = 0
    for t in range(len(bof) - 1):
        r = rec[blst[bof[t]:bof[t + 1]]]
        if gof[t] == gof[t + 1] or len(r) == 0:
            continue
        prim, sigma = r[:, oracle.GR["PRIM"]].astype(int), r[:, oracle.GR["SIGMA"]] + widen
        ox, oy = t % fr.tiles_x * tile, t // fr.tiles_x * tile
        many += len(np.unique(prim)) > rows
        x, y = r[:, oracle.GR["MUX"]] - 0.5 - ox, r[:, oracle.GR["MUY"]] - 0.5 - oy
        worst = 0
        for by in range(0, tile, 8):
            for bx in range(0, tile, 8):
                on = np.ones(len(r), bool)
                if tile > 8:
                    on = ((np.floor(x - sigma) - 1 <= bx + 7) & (np.ceil(x + sigma) + 1 >= bx) &
                          (np.floor(y - sigma) - 1 <= by + 7) & (np.ceil(y + sigma) + 1 >= by)) | ~(sigma < 2 * tile)
                worst = max(worst, len(np.unique(prim[on])))
        counted += worst > rows
    return counted, many


@pytest.mark.parametrize("tile,batch,rows", [(8, 32, 8), (8, 64, 12), (16, 64, 12), (32, 64, 12)])
@pytest.mark.parametrize("P,sharpness,wh", [(120, 10.0, (72, 56)), (200, 6.0, (97, 70))])
def test_tiles_with_more_runs_than_rows(tile, batch, rows, P, sharpness, wh):
    sc = S.random_triangles(P=P, degree=2, seed=P)
    sc.sharpness[:] = np.float32(sharpness)
    cams = S.make_cameras([(0.2, -0.1, 3.0)], [wh])
    fr = oracle.Frame(sc, cams.cams[0], *wh, G.oracle_config(tile=tile))
    ref, many = expected(fr, tile, rows)
    G.log(f"[many runs] tile={tile} batch={batch}: {ref} tiles, {many} by their runs")
    assert ref == expected(fr, tile, rows, 1e-4)[0] == expected(fr, tile, rows, -1e-4)[0]  # (decided in FP32 too)
    g = G.run_gpu(sc, cams, tile=tile, batch=batch, lean=True, pair_factor=64.0, bpair_factor=64.0)
    assert g["status"] == 0 and g["counters"][8] == ref, (g["counters"], ref, many)
