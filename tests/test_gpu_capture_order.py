"""A captured training loop while a renderer, kept alive only by a reference
cycle, waits for the garbage collector: it has to be gone before the capture
begins, since freeing its pinned memory during one would invalidate it.  Automatic
collection is off throughout, so that nothing but the loop itself can collect it;
the capture's entry looks whether it has."""
import gc
import weakref

import numpy as np
import pytest

from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def test_garbage_is_collected_before_the_capture(monkeypatch):
    import torch
    from paper_2503_13961_amd.render import Renderer, scene_tensors
    from paper_2503_13961_amd.train import TrainStep
    G.log("[capture] order of the collection")
    sc, cams, _ = S.workload("tiny")
    dev = torch.device("cuda", 0)
    step = TrainStep(Renderer(0), sc.degree, scene_tensors(sc, dev), torch.from_numpy(cams.cams).to(dev),
                     np.ascontiguousarray(cams.wh, np.int32), torch.zeros((cams.num_pixels, 3), device=dev))
    events, enter = [], torch.cuda.graph.__enter__

    def entering(self):
        events.append("capture")
        return enter(self)
    monkeypatch.setattr(torch.cuda.graph, "__enter__", entering)
    gc.collect()
    gc.disable()
    try:
        abandoned = Renderer(0)
        abandoned.cycle = abandoned
        weakref.finalize(abandoned, events.append, "freed")
        del abandoned
        assert events == []
        res = step.run(2, check_every=2)
    finally:
        gc.enable()
    assert events == ["freed", "capture"]
    assert res == {"steps": 2, "recoveries": 0, "checks": 1}
