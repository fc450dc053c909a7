// The nearest boundary point of a run in FP32, and whether FP32 decides it.
// Plain arithmetic, also compiled for the host by the tests.
#pragma once
#include <math.h>

namespace bgt {

// Bound on |d/sigma in FP32 - in FP64| below 1 for the staged boundary points
// (offsets of at most a few pixels from their pixel centres, radii >=
// 3 sqrt(0.3)): FP32 rounds the stored offsets and radius, the squared distance
// and its ratio.
constexpr float kRatioBand = 4e-6f;
// Two ratios, as the roots of their FP32 squares (a few 1e-7 more), can be in
// the other order than in FP64 where they are this close.
constexpr float kTieBand = 2.0f * (kRatioBand + 5e-7f);

// The smallest t = (d/sigma)^2 of the points added, the first point that has it,
// and the next smallest.
struct ArgScan {
    float t1 = 2.0f;
    float t2 = 2.0f;
    int e1 = -1;
    __device__ __forceinline__ void add(float t, int e) {
        t2 = fminf(t2, fmaxf(t, t1));
        if (t < t1) { t1 = t; e1 = e; }
    }
    // can a point with this t be the nearer one in FP64?  Where the ratios are within
    // kTieBand, t - t1 <= kTieBand (q + q1), and (q + q1)^2 <= 2 (t + t1).
    // (A band of one width on t is, for t1 = 1e-4, a hundred times as wide on the
    // ratio: most pixels near the boundary points of a wide radius then went on
    // to FP64.)
    __device__ __forceinline__ bool near(float t) const {
        const float d = t - t1;
        return d * d <= 2.0f * kTieBand * kTieBand * (t1 + t);
    }
    __device__ __forceinline__ bool ambiguous() const { return near(t2); }
};

}  // namespace bgt
