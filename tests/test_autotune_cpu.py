"""The autotuner's candidates against the blend kernels that there are."""
import os
import re

from paper_2503_13961_amd import autotune as A

SRC = os.path.join(os.path.dirname(os.path.abspath(A.__file__)), "csrc", "bgt_blend.hip")


def test_one_candidate_per_kernel():
    table = re.search(r"#define BGT_BLEND_CONFIGS\(X\)(.*?)\n\n", open(SRC).read(), re.S).group(1)
    kernel = {(int(t), int(b)): (int(t), int(k)) for t, b, k in re.findall(r"X\((\d+), (\d+), (\d+)\)", table)}
    assert len(kernel) == 8
    timed = [kernel[c] for c in A.CANDIDATES]
    assert len(set(timed)) == len(timed) and set(timed) == set(kernel.values())

