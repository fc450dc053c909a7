"""The loss pass at the edges of its 64x20 output tiles and of the window's
5-pixel apron: views one pixel below, at and above a multiple of the tile, and
views smaller than the window, against the FP64 oracle.  Tolerances as for the
other loss tests: the window sums are taken in FP64 from the same floats, so the
loss differs by its final rounding, and the image gradient by the float maps
between the two window passes (1e-5 of its largest entry)."""
import numpy as np
import pytest

from oracle import train as OT
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wh", [[(64, 20), (63, 19), (65, 21)], [(128, 40), (129, 5), (6, 61)], [(1, 200), (200, 1), (74, 30)]])
def test_loss_at_tile_edges(wh):
    import torch
    from paper_2503_13961_amd.render import Renderer
    from paper_2503_13961_amd.train import PhotometricLoss
    G.log(f"[loss] tile edges {wh}")
    rng = np.random.default_rng(11)
    n = int(sum(w * h for w, h in wh))
    x, y = (rng.random((n, 3)).astype(np.float32) for _ in range(2))
    dev = torch.device("cuda", 0)
    op = PhotometricLoss(Renderer(0), np.array(wh, np.int32))
    loss, grad = op(torch.from_numpy(x).to(dev), torch.from_numpy(y).to(dev))
    torch.cuda.synchronize()
    for got, ref in zip(loss.cpu().numpy().astype(np.float64), OT.loss(x, y, wh)):
        assert abs(got - ref) <= 1e-6 * abs(ref) + 1e-9
    ref = OT.loss_grad(x, y, wh)
    assert np.abs(grad.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()
