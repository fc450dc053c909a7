"""Which of two boundary points is nearer in units of its radius: FP32 decides,
unless the two are too close for it (then FP64 does).  The kernels' own
decision, compiled for the host, over radii from the smallest (3 sqrt(0.3)) to
wide ones: every pair that FP32 and FP64 order differently is handed on, and a
pair that is clearly apart is not, however small its ratios."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_13961_amd", "csrc")
CODE = """
#define __device__
#define __forceinline__ inline
#include "bgt_nearest.h"
extern "C" void scan(int n, const float *a, const float *b, int *first, int *again) {
    for (int i = 0; i < n; ++i) {
        bgt::ArgScan s;
        s.add(a[i], 0);
        s.add(b[i], 1);
        first[i] = s.e1;
        again[i] = s.ambiguous() && s.near(a[i]) && s.near(b[i]);
    }
}
"""


@pytest.fixture(scope="module")
def scan(tmp_path_factory):
    d = tmp_path_factory.mktemp("nearest")
    (d / "scan.cpp").write_text(CODE)
    subprocess.check_call(["g++", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "scan.so"),
                           str(d / "scan.cpp")])
    lib = ctypes.CDLL(str(d / "scan.so"))

    def run(a, b):
        first, again = np.zeros(len(a), np.int32), np.zeros(len(a), np.int32)
        lib.scan(len(a), *(x.ctypes.data_as(ctypes.c_void_p) for x in (a, b, first, again)))
        return first, again.astype(bool)
    return run


def _points(rng, q, sigma):
    """Points at ratio q: the offset from a pixel `p` of the point's own pixel
    centre (a few pixels at most) and the radius, rounded as they are stored;
    t in FP32 and the ratio in FP64."""
    n, f = len(q), np.float32
    ang = rng.uniform(0, 2 * np.pi, n)
    x, y = q * sigma * np.cos(ang), q * sigma * np.sin(ang)
    px, py = np.rint(x + rng.uniform(-1, 1, n)), np.rint(y + rng.uniform(-1, 1, n))
    ox, oy = (x - px).astype(f), (y - py).astype(f)
    dx, dy = f(px) + ox, f(py) + oy
    d2 = (dx.astype(np.float64) ** 2 + (dy * dy).astype(np.float64)).astype(f)  # fma(dx, dx, dy dy)
    s = sigma.astype(f)
    return d2 * (f(1) / (s * s)), np.hypot(x, y) / sigma


@pytest.mark.parametrize("lo,hi", [(1.6431677, 3.0), (3.0, 60.0), (60.0, 1000.0)])
def test_fp32_hands_on_what_it_cannot_decide(scan, lo, hi):
    rng = np.random.default_rng(int(lo))
    n = 400_000
    q = np.exp(rng.uniform(np.log(1e-3), np.log(0.999), n))
    gap = np.exp(rng.uniform(np.log(1e-9), np.log(1e-5), n)) * rng.choice([-1, 1], n)
    ta, qa = _points(rng, q, rng.uniform(lo, hi, n))
    tb, qb = _points(rng, q + gap, rng.uniform(lo, hi, n))
    first, again = scan(ta, tb)
    wrong = (qa < qb) != (first == 0)
    assert wrong.any() and again[wrong].all()


@pytest.mark.parametrize("q", [0.003, 0.01, 0.1, 0.5, 0.95])
def test_ratios_clearly_apart_are_decided_in_fp32(scan, q):
    gap = 3e-5  # seven times the bound on a ratio's error
    a = np.linspace(q, 1.02 * q, 1000)
    first, again = scan((a ** 2).astype(np.float32), ((a + gap) ** 2).astype(np.float32))
    assert (first == 0).all() and not again.any()
