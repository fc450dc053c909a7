"""The loss pass at the line between its two kernels: up to 1024 output tiles a
workgroup takes the three channels side by side, beyond that after each other.
Columns one pixel wide reach the line with few pixels.  Tolerances as for the
other loss tests: window sums in FP64 from the same floats, so 1e-6 for the loss
and, from the float maps between the window passes, 1e-5 of the largest entry
for the image gradient; the loss without a gradient is the same number."""
import numpy as np
import pytest

from oracle import train as OT
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wh", [[(1, 1)], [(167, 127)], [(64, 20)] * 9 + [(3, 41)],
                                [(1, 16384), (1, 4080)], [(1, 16384), (1, 4081)], [(2, 16384), (65, 2100)]])
def test_loss_channel_groups(wh):
    import torch
    from paper_2503_13961_amd.render import Renderer
    from paper_2503_13961_amd.train import PhotometricLoss
    G.log(f"[loss] channel groups {wh[:2]} x {len(wh)}")
    rng = np.random.default_rng(13)
    n = int(sum(w * h for w, h in wh))
    x, y = (rng.random((n, 3)).astype(np.float32) for _ in range(2))
    dev = torch.device("cuda", 0)
    op = PhotometricLoss(Renderer(0), np.array(wh, np.int32))
    xt, yt = torch.from_numpy(x).to(dev), torch.from_numpy(y).to(dev)
    grad = torch.full((n, 3), float("nan"), device=dev)
    loss, _ = op(xt, yt, grad)
    loss = loss.cpu().numpy().copy()
    alone = op(xt, yt, want_grad=False)[0].cpu().numpy()
    assert np.array_equal(alone, loss)
    for got, ref in zip(loss.astype(np.float64), OT.loss(x, y, wh)):
        assert abs(got - ref) <= 1e-6 * abs(ref) + 1e-9
    ref = OT.loss_grad(x, y, wh)
    assert np.abs(grad.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()
