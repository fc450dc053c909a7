"""A captured training loop while an abandoned renderer, kept alive only by a
reference cycle, waits for the garbage collector."""
import gc

import numpy as np
import pytest

from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def test_capture_with_an_abandoned_renderer():
    import torch
    from paper_2503_13961_amd.render import Renderer, scene_tensors
    from paper_2503_13961_amd.train import TrainStep
    G.log("[capture] abandoned renderer")
    sc, cams, _ = S.workload("tiny")
    dev = torch.device("cuda", 0)
    targets = torch.zeros((cams.num_pixels, 3), device=dev)
    step = TrainStep(Renderer(0), sc.degree, scene_tensors(sc, dev), torch.from_numpy(cams.cams).to(dev),
                     np.ascontiguousarray(cams.wh, np.int32), targets)
    old = gc.get_threshold()
    gc.collect()
    gc.disable()
    try:
        abandoned = Renderer(0)
        abandoned.cycle = abandoned
        del abandoned
        gc.set_threshold(1, 1, 1)
        gc.enable()
        res = step.run(2, check_every=2)
    finally:
        gc.enable()
        gc.set_threshold(*old)
    assert res == {"steps": 2, "recoveries": 0, "checks": 1}
