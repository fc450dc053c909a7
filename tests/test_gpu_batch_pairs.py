"""At 16 and 32 px every accepted batch takes the same kernel: images in every
bit, gradients up to the order of float atomics."""
import numpy as np
import pytest

from paper_2503_13961_amd import scenes as S
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,batch", [(16, 32), (16, 128), (32, 32), (32, 128)])
def test_batches_of_larger_tiles(tile, batch):
    G.log(f"[batch] {tile}x{batch}")
    sc, cams, _ = S.workload("sphere_small")
    gi = np.sign(np.random.default_rng(3).standard_normal((cams.num_pixels, 3))) / (3 * cams.num_pixels)
    a, b = (G.run_gpu(sc, cams, tile=tile, batch=n, grad_images=gi, lean=True) for n in (64, batch))
    np.testing.assert_array_equal(a["images"], b["images"])
    for k in a["grads"]:
        assert G.grad_error(b["grads"][k], a["grads"][k]) <= 1e-5, k
