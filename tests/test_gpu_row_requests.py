"""The rows of boundary weights that the blend passes ask memory for: as many as
runs reach a block beyond the rows in LDS, also for a tile whose list is longer than
the stage, so that the pool lasts for the other tiles.  Against the same number over
the oracle's lists; the backward asks for a row of sums beside each."""
import numpy as np
import pytest

import oracle
from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def _rows_needed(fr, tile, in_lds, widen=0.0):
    """(rows beyond in_lds per block, summed; longest list; most runs in a tile)"""
    rec, (gof, _), (bof, blst) = fr.records(), fr.lists(0), fr.lists(1)
    total = longest = runs = 0
    for t in range(len(bof) - 1):
        r = rec[blst[bof[t]:bof[t + 1]]]
        if gof[t] == gof[t + 1] or len(r) == 0:
            continue
        longest = max(longest, len(r))
        prim, sigma = r[:, oracle.GR["PRIM"]].astype(int), r[:, oracle.GR["SIGMA"]] + widen
        runs = max(runs, len(np.unique(prim)))
        x = r[:, oracle.GR["MUX"]] - 0.5 - t % fr.tiles_x * tile
        y = r[:, oracle.GR["MUY"]] - 0.5 - t // fr.tiles_x * tile
        for by in range(0, tile, 8):
            for bx in range(0, tile, 8):
                on = np.ones(len(r), bool)
                if tile > 8:
                    on = ((np.floor(x - sigma) - 1 <= bx + 7) & (np.ceil(x + sigma) + 1 >= bx) &
                          (np.floor(y - sigma) - 1 <= by + 7) & (np.ceil(y + sigma) + 1 >= by)) | ~(sigma < 2 * tile)
                total += max(len(np.unique(prim[on])) - in_lds, 0)
    return total, longest, runs


@pytest.mark.parametrize("tile,batch,in_lds,stage", [(8, 32, 8, 88), (8, 64, 12, 112), (16, 64, 12, 256), (32, 64, 12, 512)])
def test_rows_asked_for(tile, batch, in_lds, stage):
    import torch
    from paper_2503_13961_amd.render import Renderer, scene_tensors
    sc = S.random_triangles(P=60, degree=2, seed=60)
    sc.sharpness[:] = np.float32(0.1)
    cams = S.make_cameras([(0.2, -0.1, 3.0)], [(97, 70)])
    fr = oracle.Frame(sc, cams.cams[0], 97, 70, G.oracle_config(tile=tile))
    need, longest, runs = _rows_needed(fr, tile, in_lds)
    G.log(f"[rows] tile={tile} batch={batch}: {need} rows, up to {longest} points and {runs} runs in a tile")
    assert longest > stage and runs <= 64 and need > 0
    assert need == _rows_needed(fr, tile, in_lds, 1e-4)[0] == _rows_needed(fr, tile, in_lds, -1e-4)[0]  # (decided in FP32 too)
    dev = torch.device("cuda", 0)
    r = Renderer(0, tile=tile, batch=batch, pair_factor=64.0, bpair_factor=64.0)
    params, camt = scene_tensors(sc, dev), torch.from_numpy(cams.cams).to(dev)
    img, state = r.forward(sc.degree, params, camt, cams.wh)
    r.backward(sc.degree, params, camt, cams.wh, img, torch.ones_like(img), state)
    o = r.layout(sc.degree, params, camt, cams.wh)["counters"]
    asked = state[o:o + 80].cpu().numpy().view(np.int64)[8:10]
    assert list(asked) == [need, 2 * need]
