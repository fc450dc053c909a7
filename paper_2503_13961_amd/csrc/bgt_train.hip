// One training step around the renderer (Sec. 3.3): the photometric loss of
// Eq. 9, L = (1 - lambda) L2 + lambda (1 - SSIM), with its image gradient,
// and the Adam update of the parameters.
//
// SSIM takes five window moments per pixel and channel (mu_x, mu_y, E[x^2],
// E[y^2], E[xy]) under an 11x11 Gaussian window, zero outside the view, in
// FP64: E[x^2] - mu_x^2 cancels, and FP64 vector arithmetic runs at the FP32
// rate on this GPU.  A workgroup owns a 64x20 output tile of one view, one
// channel at a time (or, where tiles are few, each third of it one): it stages the tile plus a 5-pixel apron in LDS, then for
// each moment sums the window rows into LDS (a thread takes eight neighbouring
// outputs from 18 staged values) and the columns from there (a thread takes
// five outputs below each other from 15).  The per-pixel SSIM and its
// derivatives with respect to the three moments that depend on the image go to
// three maps (planes per channel); the gradient pass runs the same window over
// the maps (the window is symmetric, so its transpose is itself).  Loss
// partial sums are per workgroup and reduced in a fixed order.
//
// What bounds the passes is LDS traffic and FP64 issue.  One output per thread
// read 22 staged floats and 55 doubles of row sums per pixel and channel; with
// several outputs per thread that is 20 floats and 15 doubles, and one moment's
// row sums at a time keep a workgroup in 37 KB (27 KB in the gradient pass), four
// to a CU.
#include "bgt_internal.h"

namespace bgt {

namespace {

constexpr int kWin = 11, kApron = 5;
constexpr int kThreads = 256;
constexpr int kTW = 64, kTH = 20;                                   // output tile
constexpr int kIW = kTW + 2 * kApron, kIH = kTH + 2 * kApron;       // staged region 74 x 30
constexpr int kHOut = 8;                                            // row sums per thread: neighbouring columns
constexpr int kVOut = 5;                                            // column sums per thread: rows below each other
// LDS rows: 81 floats (a wave's 8 rows x 8 column groups start at 64 distinct
// banks: 81 is 1 mod 8); 72 doubles, column 8 g + o at position 8 o + g, so that
// the row sums of neighbouring groups are stored side by side and two rows of
// them half the banks apart (in column order, 65 doubles a row, the stores met
// on an eighth of the banks)
constexpr int kSW = 81, kHW = 72;
static_assert(kHOut * kHOut == kTW, "position 8 o + g of column 8 g + o");
__device__ __forceinline__ int column_at(int p) { return p % kHOut * kHOut + p / kHOut; }  // column of position p
static_assert(kTW / kHOut * kIH <= kThreads && kTW * (kTH / kVOut) == kThreads, "one item per thread in each pass");
// Staging: wave w takes the region's rows w, w + 4, ...; lane l columns l and,
// for the last ten, 64 + l.
constexpr int kRowsPerWave = (kIH + kThreads / 64 - 1) / (kThreads / 64);
// A workgroup has CH groups of kThreads threads, each with LDS of its own: one
// group takes the three channels after each other, or three groups one channel
// each.  A call of few tiles lasts as long as the chain of barriers in one
// workgroup, which three groups cut to a third; with many tiles the CUs fill
// better with small workgroups (one of three groups holds 110 KB of LDS).  Loss and
// gradient, one group -> three: 21 tiles (167x127) 47.9 -> 30.3 us, 240 (640x480)
// 53.4 -> 36.5, 520 (800^2) 75.7 -> 74.0, 1040 121 -> 117, 1560 153 -> 161,
// 3120 271 -> 289.
constexpr int kGroupTiles = 1024;

}  // namespace

__device__ __forceinline__ int loss_view_of_tile(const LossTable &lt, int t) {
    int lo = 0, hi = lt.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (lt.tile_off[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// sum of a double over the workgroup in a fixed order (result in thread 0)
__device__ double block_sum(double v, double *red) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
    return s;
}

// The window rows of one quantity: value(row, column) of the staged region,
// eight neighbouring sums per thread into hs.
template <typename V>
__device__ __forceinline__ void window_rows(const LossTable &lt, double (&hs)[kIH][kHW], int tid, V &&value) {
    const int r = tid / (kTW / kHOut), c0 = tid % (kTW / kHOut) * kHOut;
    if (r >= kIH) return;
    double acc[kHOut];
#pragma unroll
    for (int o = 0; o < kHOut; ++o) acc[o] = 0.0;
#pragma unroll
    for (int i = 0; i < kHOut + kWin - 1; ++i) {
        const double v = value(r, c0 + i);
#pragma unroll
        for (int o = 0; o < kHOut; ++o)
            if (i - o >= 0 && i - o < kWin) acc[o] = fma(lt.taps[i - o], v, acc[o]);
    }
#pragma unroll
    for (int o = 0; o < kHOut; ++o) hs[r][o * kHOut + c0 / kHOut] = acc[o];
}

// ... and its columns: the thread's five window sums, at position tid % 64 of
// rows 5 (tid / 64) + 0..4 of the tile
__device__ __forceinline__ void window_columns(const LossTable &lt, const double (&hs)[kIH][kHW], int tid,
                                               double (&out)[kVOut]) {
    const int c = tid % kTW, r0 = tid / kTW * kVOut;
#pragma unroll
    for (int o = 0; o < kVOut; ++o) out[o] = 0.0;
#pragma unroll
    for (int i = 0; i < kVOut + kWin - 1; ++i) {
        const double v = hs[r0 + i][c];
#pragma unroll
        for (int o = 0; o < kVOut; ++o)
            if (i - o >= 0 && i - o < kWin) out[o] = fma(lt.taps[i - o], v, out[o]);
    }
    // (the sums are taken here: the compiler otherwise keeps the 15 values and
    // takes the sums where they are used, past the barriers)
#pragma unroll
    for (int o = 0; o < kVOut; ++o) asm volatile("" : "+v"(out[o]));
}

// p with its origin hidden: the compiler otherwise keeps a running pointer per
// access across the channels, over a hundred registers
template <typename T>
__device__ __forceinline__ T *hidden(T *p) {
    asm volatile("" : "+s"(p));
    return p;
}

// The staged region at (gx0, gy0) of a view of W x H whose values are `step`
// floats apart, zero outside the view: load() reads this lane's values, store()
// puts them into the stage.
struct StageRows {
    float a[kRowsPerWave], b[kRowsPerWave];
    __device__ __forceinline__ void load(const float *p, int step, int gx0, int gy0, int W, int H, int lane, int wave) {
        p = hidden(p);
        const int xa = gx0 + lane, xb = xa + 64;
        const bool ina = xa >= 0 && xa < W, inb = lane < kIW - 64 && xb < W;
#pragma unroll
        for (int n = 0; n < kRowsPerWave; ++n) {
            const int ry = wave + n * (kThreads / 64), gy = gy0 + ry;
            const bool row = ry < kIH && gy >= 0 && gy < H;
            const float *q = p + (int64_t)gy * W * step;
            a[n] = row && ina ? q[xa * step] : 0.f;
            b[n] = row && inb ? q[xb * step] : 0.f;
        }
    }
    __device__ __forceinline__ void store(float (&s)[kIH][kSW], int lane, int wave) const {
#pragma unroll
        for (int n = 0; n < kRowsPerWave; ++n) {
            const int ry = wave + n * (kThreads / 64);
            if (ry >= kIH) continue;
            s[ry][lane] = a[n];
            if (lane < kIW - 64) s[ry][64 + lane] = b[n];
        }
    }
};

// Window moments, SSIM and its derivative maps; per-workgroup sums of the
// SSIM map and of the squared error.  16 x 800^2: 0.67-0.75 -> 0.36-0.45 ms (615 MB:
// 0.12 ms at the rate of a large copy; FP64 issue alone 0.21).
template <int CH>
__global__ void __launch_bounds__(CH *kThreads) __attribute__((amdgpu_waves_per_eu(CH == 1 ? 4 : 3)))
k_ssim_fwd(LossTable lt, const float *x, const float *y, float *map_a, float *map_b, float *map_c, double *partial) {
    __shared__ float sxs[CH][kIH][kSW], sys[CH][kIH][kSW];
    __shared__ double hss[CH][kIH][kHW];
    __shared__ double red[CH * kThreads / 64];
    const int group = CH == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads);
    auto &sx = sxs[group], &sy = sys[group];
    auto &hs = hss[group];
    const int t = blockIdx.x, tid = threadIdx.x % kThreads;
    const int v = loss_view_of_tile(lt, t);
    const int W = lt.W[v], H = lt.H[v];
    const int tl = t - lt.tile_off[v], tx = tl % lt.tiles_x[v], ty = tl / lt.tiles_x[v];
    const int gx0 = tx * kTW - kApron, gy0 = ty * kTH - kApron;
    const int64_t base = lt.px_off[v], plane = lt.total_px;
    const int c0 = column_at(tid % kTW), r0 = tid / kTW * kVOut;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool grads = map_a != nullptr;  // (no gradient wanted: no maps)
    double s_ssim = 0.0, s_sq = 0.0;
#pragma unroll 1
    for (int c = group; c < 3; c += CH) {
        StageRows rx, ry;
        rx.load(x + base * 3 + c, 3, gx0, gy0, W, H, lane, wave);
        ry.load(y + base * 3 + c, 3, gx0, gy0, W, H, lane, wave);
        // (the last reads of the previous channel's stage were its row sums',
        // before the barrier that its column sums waited at)
        rx.store(sx, lane, wave);
        ry.store(sy, lane, wave);
        __syncthreads();
        const int gx = tx * kTW + c0;
#pragma unroll
        for (int o = 0; o < kVOut; ++o) {
            const double d = (double)sx[r0 + o + kApron][c0 + kApron] - (double)sy[r0 + o + kApron][c0 + kApron];
            if (gx < W && ty * kTH + r0 + o < H) s_sq = fma(d, d, s_sq);
        }
        auto moment = [&](double(&out)[kVOut], auto &&value) {
            window_rows(lt, hs, tid, value);
            __syncthreads();
            window_columns(lt, hs, tid, out);
            __syncthreads();
        };
        double mx5[kVOut], my5[kVOut], e[kVOut], B25[kVOut];
        moment(mx5, [&](int r, int i) { return (double)sx[r][i]; });
        moment(my5, [&](int r, int i) { return (double)sy[r][i]; });
        // (products of two floats are exact in FP64)
        moment(e, [&](int r, int i) { return (double)sx[r][i] * (double)sx[r][i]; });
#pragma unroll
        for (int o = 0; o < kVOut; ++o) B25[o] = e[o] - mx5[o] * mx5[o];  // sigma_x^2
        moment(e, [&](int r, int i) { return (double)sy[r][i] * (double)sy[r][i]; });
#pragma unroll
        for (int o = 0; o < kVOut; ++o) B25[o] = B25[o] + (e[o] - my5[o] * my5[o]) + kSsimC2;
        moment(e, [&](int r, int i) { return (double)sx[r][i] * (double)sy[r][i]; });
        float *const ma = hidden(map_a + c * plane + base), *const mb = hidden(map_b + c * plane + base),
                     *const mc = hidden(map_c + c * plane + base);
#pragma unroll
        for (int o = 0; o < kVOut; ++o) {
            const int gy = ty * kTH + r0 + o;
            if (gx >= W || gy >= H) continue;
            const double mx = mx5[o], my = my5[o], sxy = e[o] - mx * my;
            const double A1 = 2.0 * mx * my + kSsimC1, A2 = 2.0 * sxy + kSsimC2;
            const double B1 = mx * mx + my * my + kSsimC1, B2 = B25[o];
            // S = A1 A2 / (B1 B2); S / A1 and S / A2 need no division of their own
            const double iB = 1.0 / (B1 * B2), SA1 = A2 * iB, SA2 = A1 * iB, S = A1 * SA1;
            s_ssim += S;
            if (!grads) continue;
            const double iB1 = B2 * iB, iB2 = B1 * iB;
            // dS/dmu_x, dS/dE[x^2], dS/dE[xy] with sigma_x^2 = E[x^2] - mu_x^2, sigma_xy = E[xy] - mu_x mu_y
            const double da = 2.0 * (my * (SA1 - SA2) + mx * S * (iB2 - iB1));
            const int q = gy * W + gx;
            ma[q] = (float)da;
            mb[q] = (float)(-S * iB2);
            mc[q] = (float)(2.0 * SA2);
        }
    }
    const double a = block_sum(s_ssim, red);
    const double b = block_sum(s_sq, red);
    if (threadIdx.x == 0) {
        partial[2 * (int64_t)t] = a;
        partial[2 * (int64_t)t + 1] = b;
    }
}

// loss[0] = L, loss[1] = L2, loss[2] = SSIM, from the per-workgroup sums, by one
// workgroup of N threads with K loads in flight each (31 -> 7 us for 16 x 800^2)
template <int N, int K>
__device__ __forceinline__ void final_sums(const LossTable &lt, const double *partial, float *loss, double *red) {
    double s[K], q[K];
#pragma unroll
    for (int k = 0; k < K; ++k) s[k] = q[k] = 0.0;
    const double2 *p = (const double2 *)partial;
    for (int i = threadIdx.x; i < lt.total_tiles; i += K * N) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (i + k * N < lt.total_tiles) {
                const double2 v = p[i + k * N];
                s[k] += v.x;
                q[k] += v.y;
            }
    }
#pragma unroll
    for (int k = 1; k < K; k *= 2)
#pragma unroll
        for (int j = 0; j < K; j += 2 * k) {
            s[j] += s[j + k];
            q[j] += q[j + k];
        }
    const double S = block_sum(s[0], red);
    const double Q = block_sum(q[0], red);
    if (threadIdx.x == 0) {
        const double l2 = Q * lt.inv_n, ssim = S * lt.inv_n;
        loss[0] = (float)((1.0 - lt.lam) * l2 + lt.lam * (1.0 - ssim));
        loss[1] = (float)l2;
        loss[2] = (float)ssim;
    }
}

// (three groups: the same sums as the gradient pass takes, for a call without one)
template <int CH>
constexpr int kFinal = CH == 1 ? 1024 : CH * kThreads;
template <int CH>
constexpr int kFinalLoads = CH == 1 ? 4 : 2;
template <int CH>
__global__ void __launch_bounds__(kFinal<CH>) k_loss_final(LossTable lt, const double *partial, float *loss) {
    __shared__ double red[kFinal<CH> / 64];
    final_sums<kFinal<CH>, kFinalLoads<CH>>(lt, partial, loss, red);
}

// dL/dC = (1 - lambda) 2 (x - y) / n - lambda / n * (W*a + 2 x W*b + y W*c)
// One map at a time; the next one's values are loaded during the sums.
// 16 x 800^2: 0.49-0.55 -> 0.30-0.35 ms (738 MB: 0.15 ms at the rate of a large copy).
// With three groups the first workgroup takes the loss from the partial sums, beside
// the others (a launch less: 30.3 -> 27.5 us for the whole call at 167x127, 74.2 ->
// 71.5 at 800^2).  With one group that costs the gradient more than the launch does
// (674 -> 681 us for 16 x 800^2).
template <int CH>
__global__ void __launch_bounds__(CH *kThreads) __attribute__((amdgpu_waves_per_eu(CH == 1 ? 4 : 3)))
k_ssim_grad(LossTable lt, const float *x, const float *y, const float *map_a, const float *map_b, const float *map_c,
            float *grad, const double *partial, float *loss) {
    __shared__ float sms[CH][kIH][kSW];
    __shared__ double hss[CH][kIH][kHW];
    const int group = CH == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads);
    auto &sm = sms[group];
    auto &hs = hss[group];
    if (CH == 3 && blockIdx.x == 0) {
        final_sums<kFinal<CH>, kFinalLoads<CH>>(lt, partial, loss, &hss[0][0][0]);
        return;
    }
    const int t = CH == 3 ? blockIdx.x - 1 : blockIdx.x, tid = threadIdx.x % kThreads;
    const int v = loss_view_of_tile(lt, t);
    const int W = lt.W[v], H = lt.H[v];
    const int tl = t - lt.tile_off[v], tx = tl % lt.tiles_x[v], ty = tl / lt.tiles_x[v];
    const int gx0 = tx * kTW - kApron, gy0 = ty * kTH - kApron;
    const int64_t base = lt.px_off[v], plane = lt.total_px;
    const int c0 = column_at(tid % kTW), r0 = tid / kTW * kVOut;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    StageRows next;
    next.load(map_a + group * plane + base, 1, gx0, gy0, W, H, lane, wave);
    const int gx = tx * kTW + c0, gy0o = ty * kTH + r0;
    float res[3 / CH][kVOut];  // (written together at the end: 12 bytes per pixel)
#pragma unroll
    for (int i = 0; i < 3 / CH; ++i) {
        const int c = group + i;
        float xv[kVOut], yv[kVOut];
        {
            const float *const xp = hidden(x + base * 3 + c), *const yp = hidden(y + base * 3 + c);
#pragma unroll
            for (int o = 0; o < kVOut; ++o) {
                const bool in = gx < W && gy0o + o < H;
                const int q = in ? ((gy0o + o) * W + gx) * 3 : 0;
                xv[o] = xp[q];
                yv[o] = yp[q];
            }
        }
        double w[3][kVOut];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            next.store(sm, lane, wave);
            __syncthreads();
            const float *map = k == 0 ? map_b : (k == 1 ? map_c : map_a);
            if (k < 2 || i + 1 < 3 / CH) next.load(map + (c + (k == 2)) * plane + base, 1, gx0, gy0, W, H, lane, wave);
            window_rows(lt, hs, tid, [&](int r, int j) { return (double)sm[r][j]; });
            __syncthreads();
            window_columns(lt, hs, tid, w[k]);
            // (the stage is free from the barrier above on; hs is written
            // again only after the barrier that follows the next fill)
        }
#pragma unroll
        for (int o = 0; o < kVOut; ++o) {
            const double a = xv[o], b = yv[o];
            res[i][o] = (float)((1.0 - lt.lam) * 2.0 * (a - b) * lt.inv_n -
                                lt.lam * lt.inv_n * (w[0][o] + 2.0 * a * w[1][o] + b * w[2][o]));
        }
    }
    float *const gp = grad + base * 3;
#pragma unroll
    for (int o = 0; o < kVOut; ++o) {
        if (gx >= W || gy0o + o >= H) continue;
        float *q = gp + (int64_t)((gy0o + o) * W + gx) * 3 + group;
#pragma unroll
        for (int i = 0; i < 3 / CH; ++i) q[i] = res[i][o];
    }
}

template <int CH>
static void loss_passes(const LossTable &lt, const float *x, const float *y, float *loss, float *grad, float *maps,
                        double *partial, hipStream_t s) {
    const int64_t n = 3 * (int64_t)lt.total_px;
    float *ma = maps, *mb = maps + n, *mc = maps + 2 * n;
    hipLaunchKernelGGL(k_ssim_fwd<CH>, dim3(lt.total_tiles), dim3(CH * kThreads), 0, s, lt, x, y,
                       grad ? ma : nullptr, mb, mc, partial);
    if (CH == 1 || !grad)
        hipLaunchKernelGGL(k_loss_final<CH>, dim3(1), dim3(kFinal<CH>), 0, s, lt, (const double *)partial, loss);
    if (grad)
        hipLaunchKernelGGL(k_ssim_grad<CH>, dim3(lt.total_tiles + (CH == 3)), dim3(CH * kThreads), 0, s, lt, x, y,
                           (const float *)ma, (const float *)mb, (const float *)mc, grad, (const double *)partial,
                           loss);
}

hipError_t launch_loss(const LossTable &lt, const float *x, const float *y, float *loss, float *grad, float *maps,
                       double *partial, hipStream_t s) {
    if (lt.total_tiles <= kGroupTiles)
        loss_passes<3>(lt, x, y, loss, grad, maps, partial, s);
    else
        loss_passes<1>(lt, x, y, loss, grad, maps, partial, s);
    return hipGetLastError();
}

void loss_tiles(int W, int H, int *tiles_x, int *tiles) {
    *tiles_x = (W + kTW - 1) / kTW;
    *tiles = *tiles_x * ((H + kTH - 1) / kTH);
}

// ------------------------------------------------------------------- L1

__global__ void __launch_bounds__(kThreads) k_l1_cotangent(int64_t n, const float *x, const float *y, float scale,
                                                           float *g) {
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        const float d = x[i] - y[i];
        g[i] = d > 0.f ? scale : (d < 0.f ? -scale : 0.f);
    }
}

hipError_t launch_l1(int64_t n, const float *x, const float *y, float scale, float *g, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + kThreads - 1) / kThreads;
    blocks = blocks > 8192 ? 8192 : blocks;
    hipLaunchKernelGGL(k_l1_cotangent, dim3((unsigned)blocks), dim3(kThreads), 0, s, n, x, y, scale, g);
    return hipGetLastError();
}

// ------------------------------------------------------------------- Adam

// One Adam update (Kingma and Ba, Algorithm 1) over every group, at step
// *step + 1; FP64 arithmetic, moments stored as float.
__global__ void __launch_bounds__(kThreads) k_adam(AdamTable at, double b1, double b2, double eps,
                                                   const int32_t *step) {
    const int64_t total = at.off[at.n];
    const int t1 = step[0] + 1;
    const double bc1 = 1.0 - pow(b1, (double)t1), bc2 = 1.0 - pow(b2, (double)t1);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        int g = 0;
        while (i >= at.off[g + 1]) ++g;
        const int64_t j = i - at.off[g];
        const double gr = at.grad[g][j];
        const double m = b1 * (double)at.m[g][j] + (1.0 - b1) * gr;
        const double v = b2 * (double)at.v[g][j] + (1.0 - b2) * gr * gr;
        at.m[g][j] = (float)m;
        at.v[g][j] = (float)v;
        at.param[g][j] = (float)((double)at.param[g][j] - at.lr[g] * (m / bc1) / (sqrt(v / bc2) + eps));
    }
}

__global__ void k_step_advance(int32_t *step) {
    if (threadIdx.x == 0) step[0] += 1;
}

hipError_t launch_adam(const AdamTable &at, double b1, double b2, double eps, int32_t *step, hipStream_t s) {
    const int64_t total = at.off[at.n];
    if (total > 0) {
        int64_t blocks = (total + kThreads - 1) / kThreads;
        if (blocks > 2048) blocks = 2048;
        hipLaunchKernelGGL(k_adam, dim3((unsigned)blocks), dim3(kThreads), 0, s, at, b1, b2, eps,
                           (const int32_t *)step);
    }
    hipLaunchKernelGGL(k_step_advance, dim3(1), dim3(64), 0, s, step);
    return hipGetLastError();
}

}  // namespace bgt
