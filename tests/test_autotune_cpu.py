"""The autotuner's candidates against the blend kernels that there are, and the
cache key against the library that a choice was timed on."""
import os
import re

import numpy as np

from paper_2503_13961_amd import autotune as A

SRC = os.path.join(os.path.dirname(os.path.abspath(A.__file__)), "csrc", "bgt_blend.hip")


def test_one_candidate_per_kernel():
    table = re.search(r"#define BGT_BLEND_CONFIGS\(X\)(.*?)\n\n", open(SRC).read(), re.S).group(1)
    kernel = {(int(t), int(b)): (int(t), int(k)) for t, b, k in re.findall(r"X\((\d+), (\d+), (\d+)\)", table)}
    assert len(kernel) == 8
    timed = [kernel[c] for c in A.CANDIDATES]
    assert len(set(timed)) == len(timed) and set(timed) == set(kernel.values())


def test_cache_key_names_the_library(tmp_path, monkeypatch):
    import torch
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: type("P", (), {"gcnArchName": "gfx950:x"}))
    wh = np.array([[64, 48]], np.int32)
    keys = []
    for content in (b"one", b"two", b"one"):
        lib = tmp_path / "lib.so"
        lib.write_bytes(content)
        monkeypatch.setattr("paper_2503_13961_amd.native.LIB_PATH", str(lib))
        keys.append(A.shape_key(2, 100, wh))
    assert keys[0] != keys[1] and keys[0] == keys[2]
