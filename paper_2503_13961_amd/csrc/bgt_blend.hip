// Discontinuity-aware alpha blending (Sec. 3.2, Eq. 6-8) and its backward
// pass (Supplementary Sec. C) on gfx950.
//
// One workgroup renders one TSxTS tile; each wave owns an 8x8 pixel block,
// each lane one of its pixels and each 16-lane row a 4x4 sub-block.  The
// tile's boundary points (sorted by primitive id) are staged in LDS and split
// into runs of equal id.  For every run r that reaches its block a wave builds
// a row
//     gamma*_r(q) = min over the run's points b of min(2^(|q-b|/sigma_b - 1), 1)
// of its 64 pixels, every lane its own pixel's value, and keeps the weight w of
// Eq. 6 it gives a Gaussian of the run there, so the blend loop reads w instead
// of searching boundary points per (pixel, Gaussian) pair; a Gaussian of
// primitive g finds its run by binary search over the run ids.
// Gaussians are then composited front to back in LDS-staged batches.  A
// ballot per sub-block marks the batch entries that can reach it, and each
// row walks its own mask, so the four rows of a wave work on four (possibly
// different) Gaussians per step; a Gaussian that misses a sub-block costs that
// sub-block nothing.
#include <type_traits>

#include "bgt_internal.h"
#include "bgt_nearest.h"
#include "bgt_wave.h"

namespace bgt {

// Per-wave rows of w (Eq. 6) in LDS (forward, backward; the backward sums dl/dw
// of each in registers), boundary points staged at once and entries of the run
// table.  Rows beyond those go to memory the binning has left unused
// (RowPool), a longer list is staged in chunks, and only primitives beyond the
// run table, or rows the pool has no room for, are searched per pixel and
// Gaussian.  The budget sets how many waves share a SIMD: at 8 px (one wave
// per workgroup) under 6.25 KB with 32-entry batches; `batch` 64 takes the
// variant with more points and rows for scenes with more runs per tile.  The 2000-patch sphere at
// 16 x 800^2 has at most 12 runs and 91 points in an 8 px tile (mean 2.6
// runs); in the 50,000-patch sphere at 32 x 1024x768 a third of the tiles have
// more than 12 runs (up to 33) and up to 120 points.  LDS is allocated in units
// of 1280 bytes: 5888 bytes (8 px, batch 32) and 7664 (batch 64) leave room for
// 25 and 21 workgroups on a CU.  Searching the runs
// without a row per pixel and Gaussian bound such scenes: the forward of 50,000
// patches took 4.16 ms and takes 1.91, that of 8000 cubic patches at 1000x1000
// and 16 px (rows per tile then, twelve in all) 2.25 and 0.155 ms, that of 64
// patches at 128x128 and 16 px 2.37 and 0.122 ms.
template <int TS, int K>
struct BlendDims {
    static constexpr int NW = TS * TS / 64;                          // waves
    // Gaussians staged per batch of a wave: every wave stages the tile's list
    // for its own 8x8 block, whichever the tile size, and goes through it at its
    // own pace.  (The waves of a 16 or 32 px tile shared batches staged by
    // one of them, with two barriers each, at which they waited for the
    // slowest: forward of 2000 patches' lattice in 8 views of 800x800 0.96 ->
    // 0.77 ms, 8000 cubic patches at 1000x1000 0.245 -> 0.19 ms; 32 px tiles,
    // four views of 800x800, 1.34 -> 0.57 ms; 0.43, 0.155 and 0.50 with the tile
    // order and own_prims.)  64 entries fill the loaders' lanes (16 px, 32
    // entries: 0.80 against 0.77 ms for the lattice), 32 keep a fifth wave per SIMD
    // at 8 px and in the backward.
    static constexpr int KI_FWD = TS == 8 ? 32 : 64;
    static constexpr int KI_BWD = 32;
    static constexpr int CAP = TS >= 32 ? 512 : (TS >= 16 ? 256 : (K > 32 ? 112 : 88));
    static constexpr int NR = TS >= 16 ? 128 : (K > 32 ? 96 : 64);
    static constexpr int RM_FWD = TS >= 16 ? 12 : (K > 32 ? 12 : 8);
    static constexpr int RM_BWD = TS >= 16 ? 12 : (K > 32 ? 12 : 8);
};

// Thread layout: wave w owns the 8x8 block (w % SPR, w / SPR); lane l of it
// the pixel (4 (q & 1) + (i & 3), 4 (q >> 1) + (i >> 2)) of that block, with
// q = l / 16 its row (4x4 sub-block) and i = l % 16.
template <int TS>
struct TileGeom {
    static constexpr int NT = TS * TS;
    static constexpr int SPR = TS / 8;  // 8x8 blocks per tile row
    __device__ static __forceinline__ void local_xy(int tid, int &lx, int &ly) {
        const int wave = tid >> 6, q = (tid >> 4) & 3, i = tid & 15;
        lx = (wave % SPR) * 8 + (q & 1) * 4 + (i & 3);
        ly = (wave / SPR) * 8 + (q >> 1) * 4 + (i >> 2);
    }
};

// Boundary staging shared by forward and backward.  Boundary point e sits at
// pixel (bix, biy) (tile-relative) plus the offset (bdx, bdy) of its projected
// position from that pixel's centre; distances to pixel (x, y) are
// (x - bix) - bdx etc., an exact integer minus one float, so every value
// depends only on the point and the pixel, never on the tile.
template <int TS, int K, int RM_>
struct BoundaryLds {
    using D = BlendDims<TS, K>;
    static constexpr int CAP = D::CAP, NR = D::NR, NW = D::NW, RM = RM_;
    float4 pt[CAP];      // (bdx, bdy, 1 / sigma^2, bix | biy << 16 as an int16 pair)
    float sigma[CAP];
    int run_prim[NR];
    int run_start[NR + 1];  // first point of each run, a position in the tile's list
    uint8_t row_of[NW > 1 ? NW : 1][NW > 1 ? NR : 1];  // each wave's row of a run (255: the run does not reach its block)
    int run_mask[NW > 1 ? NR : 1];  // the waves that the staged points of a run reach
    int ws[NW + 1];                 // the scan's wave totals; last: a wave has found more rows than fit LDS
    int nmap[NW];                   // rows each wave has memory for
    float map[NW * RM][64];         // rows of w
    static_assert(NR <= 128, "row indices fit the entries' signed bytes");
};

// Memory for gamma* rows beyond the LDS ones: the key arrays of the two tile
// lists, which nothing reads after the sort, as rows of 64 floats handed out by
// a counter that each pass starts at zero.  A pass whose rows do not fit falls
// back to the per-pixel search for the rest.
struct RowPool {
    float *a, *b;
    int64_t na, nb;  // rows
    unsigned long long *next;
};

// n consecutive rows (called by a whole wave), null when they do not fit
__device__ __forceinline__ float *pool_rows(const RowPool &P, int n, int lane) {
    int lo = 0, hi = 0;
    if (lane == 0) {
        const unsigned long long v = atomicAdd(P.next, (unsigned long long)n);
        lo = (int)(unsigned)v;
        hi = (int)(v >> 32);
    }
    const int64_t r = ((int64_t)__builtin_amdgcn_readfirstlane(hi) << 32) | (unsigned)__builtin_amdgcn_readfirstlane(lo);
    if (r + n <= P.na) return P.a + r * 64;
    const int64_t rb = r - P.na;
    if (rb >= 0 && rb + n <= P.nb) return P.b + rb * 64;
    return nullptr;
}

// Lane masks: the ballot of one comparison is the comparison itself, while
// that of a combined flag costs a select and another comparison, so combined
// conditions are formed from masks by scalar instructions.
typedef unsigned long long LaneMask;
__device__ __forceinline__ LaneMask lanes(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ bool in_mask(LaneMask m) { return __builtin_amdgcn_inverse_ballot_w64(m); }  // (m wave-uniform)
__device__ __forceinline__ bool any_lane(bool b) { return lanes(b) != 0ull; }
__device__ __forceinline__ bool all_lanes(bool b) { return !any_lane(!b); }

// A wave's batch.  A staged Gaussian's mean is kept as (g - w0) + delta, where
// g is the Gaussian's own pixel, w0 the origin of the wave's 8x8 block and delta
// the mean's offset from g's centre: one rounding that does not depend on
// the tile size.
template <int KI>
struct BatchLds {
    struct MP {
        float2 m;
        int2 pr;  // primitive, row code: a row index, kNoRow (the run has no point near the block: gamma* = 1) or kSearch
    };
    // (three 16-byte records: one address serves every read of an entry)
    MP mp[KI];
    float4 e[KI];  // conic in exponent form kE (a, 2b, c), opacity
    float4 c[KI];  // colour; w: free (the backward's record index)
};
constexpr int kNoRow = -1, kSearch = -2;

// |q - b| has its cone point at d = 0, where the subgradient taken is 0; a
// boundary point on its own pixel centre (every boundary pixel of a planar
// patch) lands there up to rounding, so distances below kDKink pixels count
// as 0 for the position gradient
constexpr float kDKink = 1e-6f;
// Bound on |(d/sigma)^2 in FP32 - in FP64| below 1: d/sigma is within kRatioBand, its
// square within twice that, and the products add a few 1e-7.
constexpr float kTBand = 9e-6f;
// A point is in range where d/sigma < 1; where (d/sigma)^2 in FP32 is within
// 2 kTBand of 1 the ratio itself, the FP32 quotient, decides that.
constexpr float kTIn = 1.0f - 2.0f * kTBand, kTOut = 1.0f + 2.0f * kTBand;

// -log2(e)/2: G = exp(-d^T Q d / 2) = 2^(kE d^T Q d)
constexpr float kE = -0.5f * 1.44269504088896341f;

// 2^e for the support exponent e in [log2(g_min), 0]: the hardware exp2
// (no denormal range reduction is needed there).  Forward and backward use
// this one function, so the backward's replay reproduces the forward's
// transmittance bit for bit.
__device__ __forceinline__ float support_exp2(float e) { return __builtin_amdgcn_exp2f(e); }

// The primitives of a block's pixels, their ids mod 32 as bits: an entry of another
// primitive without a row has w = 0 on the whole block and is left out of the
// batch's mask.  (A primitive that shares the bit of one of them stays in and is
// dropped at its pixels.)  Lists of wide Gaussians are mostly such entries, and every
// wave walked them: one 256x256 view of 64 patches, Gaussians of 20 px, 16 px tiles,
// backward 2.97 -> 1.96 ms (2.51 with batches shared by the waves of a tile),
// forward 2.98 -> 2.01; lattice of 2000 patches in 8 views of 800x800, step 2.62 ->
// 2.14 ms; 16 views of 800x800 at 8 px 3.34 -> 3.30.  (With 64 bits the lattice's forward
// is 2 % faster and those of 16 views and of 20,000 cubic patches 0.5 and 1 % slower: a
// bit of 64 takes five instructions where one of 32 takes one.)
__device__ __forceinline__ unsigned own_prims(int h) {  // h: each lane's primitive, -1: none
    return wave_or(h >= 0 ? 1u << (h & 31) : 0u);
}

// run index of primitive g among the tile's runs, -1 when absent
__device__ __forceinline__ int find_run(const int *run_prim, int n_runs, int g) {
    int lo = 0, hi = n_runs - 1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int pm = run_prim[mid];
        if (pm == g) return mid;
        if (pm < g) lo = mid + 1; else hi = mid - 1;
    }
    return -1;
}

// |(dx, dy)| and its square with an explicit rounding sequence, so every code
// path that evaluates a boundary distance produces the same bits
__device__ __forceinline__ float bdist2(float dx, float dy) { return __fmaf_rn(dx, dx, __fmul_rn(dy, dy)); }
__device__ __forceinline__ float bdist(float dx, float dy) { return sqrtf(bdist2(dx, dy)); }
__device__ __forceinline__ float inv_sigma2(float sigma) { return __fdiv_rn(1.0f, __fmul_rn(sigma, sigma)); }

// gamma(d; sigma) = min(2^(d/sigma - 1), 1)  (Eq. 7)
__device__ __forceinline__ float gamma_fn(float d, float sigma) {
    // (the hardware exp2: no denormal range below its argument's -1)
    const float g = __builtin_amdgcn_exp2f(__fsub_rn(__fdiv_rn(d, sigma), 1.0f));
    return g < 1.0f ? g : 1.0f;
}

// A boundary point as staged, from its record
__device__ __forceinline__ float4 boundary_point(const StatePtrs &st, int bpix, int ox, int oy, int &prim, float &sigma) {
    const float4 r0 = st.rec[(int64_t)bpix * 4];
    const float4 r2 = st.rec[(int64_t)bpix * 4 + 2];
    const int a = __float_as_int(r2.w);  // the record's pixel
    prim = __float_as_int(r2.y);
    sigma = r2.z;
    return make_float4(r0.x, r0.y, inv_sigma2(r2.z), __int_as_float(pack16(lo16(a) - ox, hi16(a) - oy)));
}
// d^2 and (d/sigma)^2 from tile-relative pixel (x, y) to a staged point
__device__ __forceinline__ float point_d2(const float4 &p, int x, int y) {
    const int b = __float_as_int(p.w);
    return bdist2((float)(x - lo16(b)) - p.x, (float)(y - hi16(b)) - p.y);
}
__device__ __forceinline__ float point_t(const float4 &p, int x, int y) { return __fmul_rn(point_d2(p, x, y), p.z); }

// w of Eq. 6 from gamma*: on pixels of the Gaussian's own primitive gamma*,
// elsewhere 1 - gamma*
__device__ __forceinline__ float weight(float gam, bool own) { return own ? gam : 1.0f - gam; }

// The boundary point the gradient of gamma* goes to (Suppl. Sec. C, dl/db):
// the minimiser of d/sigma among the points with d/sigma < 1, the lowest list
// (raster) index among exactly equal ratios.  The FP32 pass finds the smallest
// t = (d/sigma)^2 and the first point attaining it; when another point's ratio
// is too close for FP32 to tell (ArgScan::near), the order is decided again on the
// FP64 records of the points that close, which the generation pass keeps for
// every boundary point, so the choice is the one exact arithmetic makes.

// d/sigma in FP64 from pixel (x, y) to the boundary point of record bpix,
// whose pixel is (bx, by) (same frame as x, y)
__device__ __forceinline__ double ratio64(const StatePtrs &st, int bpix, int x, int y, int bx, int by) {
    const double *b = st.brec64 + (int64_t)bpix * 3;
    const double dx = (double)(x - bx) - b[0], dy = (double)(y - by) - b[1];
    return sqrt(dx * dx + dy * dy) / b[2];
}

// first entry of the tile's list with primitive >= g
__device__ __forceinline__ int first_of_prim(const StatePtrs &st, int bs0, int bc, int g) {
    int lo = 0, hi = bc;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const int pm = __float_as_int(st.rec[(int64_t)st.b_list[bs0 + mid] * 4 + 2].y);
        if (pm < g) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// The entry of the tile's list, among [e0, e1), that the gradient of gamma*
// goes to at tile pixel (lx, ly) (-1: none in range), with gamma* itself in
// *gam when asked for.  Entries below `staged` are read from LDS, the others
// from their records.
template <typename BL>
__device__ __forceinline__ int arg_min(const BL &B, const StatePtrs &st, int bs0, int e0, int e1, int staged, int lx,
                                       int ly, int ox, int oy, float *gam) {
    ArgScan a;
    int pm;
    float sg;
    for (int e = e0; e < e1; ++e) {
        const float4 p = e < staged ? B.pt[e] : boundary_point(st, (int)st.b_list[bs0 + e], ox, oy, pm, sg);
        a.add(point_t(p, lx, ly), e);
    }
    if (gam) {
        *gam = 1.0f;
        if (a.t1 < kTOut) {
            const float4 p = boundary_point(st, (int)st.b_list[bs0 + a.e1], ox, oy, pm, sg);
            *gam = gamma_fn(sqrtf(point_d2(p, lx, ly)), sg);
        }
    }
    if (!(a.t1 < kTOut)) return -1;
    if (a.t1 + 2.0f * kTBand >= kTIn) {
        // (rare) a near-tie can lie out of range: the points in range by their FP32
        // ratios, near-ties of those in FP64
        float q1 = 2.0f, q2 = 2.0f;
        int first = -1, arg = -1;
        for (int pass = 0; pass < 2; ++pass) {
            double rb = 2.0;
            for (int e = e0; e < e1; ++e) {
                const int bpix = (int)st.b_list[bs0 + e];
                const float4 p = boundary_point(st, bpix, ox, oy, pm, sg);
                const float q = __fdiv_rn(sqrtf(point_d2(p, lx, ly)), sg);
                if (!(q < 1.0f)) continue;
                if (pass == 0) {
                    if (q < q1) { q2 = q1; q1 = q; first = e; }
                    else if (q < q2) q2 = q;
                } else if (q <= q1 + 2.0f * kRatioBand) {
                    const int b = __float_as_int(p.w);
                    const double x = ratio64(st, bpix, lx, ly, lo16(b), hi16(b));
                    if (x < rb) { rb = x; arg = e; }
                }
            }
            if (pass == 0 && (first < 0 || q2 - q1 > 2.0f * kRatioBand)) return first;
        }
        return arg;
    }
    if (!a.ambiguous()) return a.e1;
    double rb = 2.0;
    int arg = -1;
    for (int e = e0; e < e1; ++e) {
        const int bpix = (int)st.b_list[bs0 + e];
        const float4 p = boundary_point(st, bpix, ox, oy, pm, sg);
        const float t = point_t(p, lx, ly);
        if (!a.near(t)) continue;
        const int b = __float_as_int(p.w);
        const double q = ratio64(st, bpix, lx, ly, lo16(b), hi16(b));
        if (q < rb) { rb = q; arg = e; }
    }
    return arg;
}

// The same for primitive g when it has no row (run table or pool full): its
// part of the list is taken from the table, or found first.
template <typename BL>
__device__ __forceinline__ int search_prim(const BL &B, const StatePtrs &st, int bs0, int bc, int g, int n_runs, int lx,
                                           int ly, int ox, int oy, float *gam) {
    const int r = find_run(B.run_prim, n_runs, g);
    const int e0 = r >= 0 ? B.run_start[r] : first_of_prim(st, bs0, bc, g);
    const int e1 = r >= 0 ? B.run_start[r + 1] : first_of_prim(st, bs0, bc, g + 1);
    return arg_min(B, st, bs0, e0, e1, bc <= BL::CAP ? bc : 0, lx, ly, ox, oy, gam);
}

// What a wave knows of its tile's runs after build_rows
struct RowInfo {
    int n_runs;     // runs in the table
    bool many;      // the list has more
    int nrow;       // rows this wave uses (LDS rows first)
    bool far;       // an entry's row can lie outside LDS, or be missing
    bool search;    // ... be missing: its primitive is searched per pixel
    float *extra;   // rows from RM on, 64 floats each (null: none)
};

// 8x8 blocks of the tile (bit w: wave w's) that a point's disc can reach, one
// pixel of margin each side; all of them for a radius that is not finite or
// exceeds two tiles.
template <int TS>
__device__ __forceinline__ int blocks_reached(const float4 &p, float sigma) {
    constexpr int SPR = TS / 8;
    if (!(sigma < (float)(2 * TS))) return (int)((1ull << (SPR * SPR)) - 1ull);
    const int b = __float_as_int(p.w);
    const float x = (float)lo16(b) + p.x, y = (float)hi16(b) + p.y;
    const int x0 = max((int)floorf(x - sigma) - 1, 0) >> 3, x1 = min((int)ceilf(x + sigma) + 1, TS - 1) >> 3;
    const int y0 = max((int)floorf(y - sigma) - 1, 0) >> 3, y1 = min((int)ceilf(y + sigma) + 1, TS - 1) >> 3;
    if (x0 > x1 || y0 > y1) return 0;
    const int row = ((2 << x1) - 1) & ~((1 << x0) - 1);
    int m = 0;
#pragma unroll
    for (int r = 0; r < SPR; ++r)
        if (r >= y0 && r <= y1) m |= row << (r * SPR);
    return m;
}

// Stages the tile's boundary points, finds the runs of equal primitive id and
// builds each wave's rows of w.  Every lane takes the minimum of t over a
// run's points at its own pixel, a dozen instructions per point: scattering each
// point over the pixels of its disc by LDS atomics took a division, a square
// root and an exponential per (point, pixel) instead of one per (run, pixel)
// (16 x 800^2 forward: 0.98 -> 0.78 ms; 0.75 now).
// A list longer than the stage is taken in chunks: only the last run of one can
// go on in the next, with the smallest t so far, so that gamma* is that of the point
// of smallest t over the whole list, as arg_min takes it.  Such a list is gone
// through twice, the first time to number the runs that reach each block: rows are
// asked for by that number.  (Asking for as many as the run table has, 116 a wave
// and twice that in the backward, emptied the pool, and the tiles that came too late
// searched per pixel: 2000 patches of sharpness 0.3 in four views of 800x800, 16 px
// tiles, forward 20.0 -> 1.25 ms, backward 37.6 -> 3.9; 1620 patches in five views of
// 151x188, backward 0.25 to 0.49 from call to call -> 0.24.)
// DG: a second row of zeros per extra row (the backward's dl/dgamma* sums), after the
// gamma* ones.
template <int TS, int K, bool DG, typename BL>
__device__ __forceinline__ RowInfo build_rows(BL &B, const StatePtrs &st, const RowPool &pool, int bs0, int bc, int ox,
                                              int oy, int lx, int ly, int h) {
    constexpr int NW = BL::NW, NR = BL::NR, CAP = BL::CAP, RM = BL::RM, NT = TS * TS;
    const int tid = threadIdx.x, lane = tid & 63, wave = NW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const unsigned long long below = (1ull << lane) - 1ull;
    RowInfo R = {0, false, 0, false, false, nullptr};
    int nr = 0, nmap = RM;  // runs so far; rows with memory
    int r_last = -1;        // the run taken last, its smallest t and the gamma of that point at this pixel
    float t_last = 2.0f, g_last = 1.0f;
    if (NW > 1 && !DG && tid == 0) B.ws[NW] = 0;
    if (bc == 0) {
        if (tid < NW) B.nmap[tid] = RM;
        __syncthreads();
        return R;
    }
    const int first_turn = bc > CAP ? 0 : 1;
    for (int turn = first_turn; turn < 2; ++turn, nr = 0)
    for (int base = 0; base < bc; base += CAP) {
        const int n = min(CAP, bc - base), first = max(nr - 1, 0);
        if (base > 0 || turn > first_turn) __syncthreads();  // every wave is done with the last chunk
        if constexpr (NW > 1) {
            for (int i = tid; i < NR; i += NT) {
                B.run_mask[i] = 0;
                if (base == 0 && turn == first_turn)
                    for (int w = 0; w < NW; ++w) B.row_of[w][i] = 255;
            }
            __syncthreads();
        }
        for (int b0 = 0; b0 < n; b0 += NT) {
            const int e = b0 + tid;
            const bool in = e < n;
            int prim = -1, before = -1;
            float sigma = 0.f;
            float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
            if (in) {
                const int bpix = (int)st.b_list[bs0 + base + e];
                p = boundary_point(st, bpix, ox, oy, prim, sigma);
                B.pt[e] = p;
                B.sigma[e] = sigma;
                // the entry before a wave's first (the others' are the lane below's)
                if (lane == 0 && base + e > 0)
                    before = __float_as_int(st.rec[(int64_t)st.b_list[bs0 + base + e - 1] * 4 + 2].y);
            }
            const int up = __shfl_up(prim, 1, 64);
            if (lane != 0) before = up;
            const bool f = in && (base + e == 0 || prim != before);
            const unsigned long long fm = __ballot(f);
            int idx = nr + (int)__popcll(fm & below) + (f ? 1 : 0) - 1;  // this point's run
            if constexpr (NW > 1) {
                if (lane == 0) B.ws[wave] = (int)__popcll(fm);
                __syncthreads();
                int tot = 0;
                for (int w = 0; w < NW; ++w) {
                    if (w < wave) idx += B.ws[w];
                    tot += B.ws[w];
                }
                __syncthreads();
                nr += tot;
                if (in && idx >= 0 && idx < NR) atomicOr(&B.run_mask[idx], blocks_reached<TS>(p, sigma));
            } else {
                nr += (int)__popcll(fm);
            }
            if (f && idx <= NR) {
                B.run_start[idx] = base + e;
                if (idx < NR) B.run_prim[idx] = prim;
            }
        }
        nr = __builtin_amdgcn_readfirstlane(nr);
        if (tid == 0 && nr <= NR) B.run_start[nr] = base + n;
        R.n_runs = min(nr, NR);
        R.many = nr > NR;
        __syncthreads();
        // rows of this chunk's runs: at 8 px every listed run reaches the
        // tile and run r takes row r; otherwise each wave numbers the runs
        // that reach its block
        if constexpr (NW > 1) {
            for (int r0 = first; r0 < R.n_runs; r0 += 64) {
                const int r = r0 + lane;
                const bool take = r < R.n_runs && ((B.run_mask[r] >> wave) & 1) && B.row_of[wave][r] == 255;
                const unsigned long long tm = __ballot(take);
                if (take) B.row_of[wave][r] = (uint8_t)(R.nrow + (int)__popcll(tm & below));
                R.nrow += (int)__popcll(tm);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            R.nrow = max(R.nrow, R.n_runs);
        }
        if (turn == 0) continue;
        if (base == 0) {
            const int more = R.nrow - RM;
            if (more > 0) {
                R.extra = pool_rows(pool, DG ? 2 * more : more, lane);
                if (R.extra) {
                    nmap = RM + more;
                    if constexpr (DG)
                        for (int i = 0; i < more; ++i) R.extra[(int64_t)(more + i) * 64 + lane] = 0.f;
                }
            }
        }
        for (int r = first; r < R.n_runs; ++r) {
            int row = r;
            if constexpr (NW > 1) {
                row = __builtin_amdgcn_readfirstlane((int)B.row_of[wave][r]);
                if (row == 255 || !((__builtin_amdgcn_readfirstlane(B.run_mask[r]) >> wave) & 1)) continue;
            }
            if (row >= nmap) continue;
            const int rs = __builtin_amdgcn_readfirstlane(B.run_start[r]), re = __builtin_amdgcn_readfirstlane(B.run_start[r + 1]);
            const int s0 = max(rs - base, 0), s1 = min(re - base, n);
            if (s0 >= s1) continue;
            // (a run that the last chunk broke off goes on from its smallest t)
            float t = r == r_last ? t_last : 2.0f, g = r == r_last ? g_last : 1.0f;
            int em = -1;
            for (int e = s0; e < s1; e += 4) {  // (four reads in flight; a short run's last point is taken again)
                float4 p[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = B.pt[min(e + i, s1 - 1)];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float ti = point_t(p[i], lx, ly);
                    const bool less = ti < t;
                    em = less ? min(e + i, s1 - 1) : em;
                    t = less ? ti : t;
                }
            }
            if (em >= 0 && t < kTOut) g = gamma_fn(sqrtf(point_d2(B.pt[em], lx, ly)), B.sigma[em]);  // (at most 1)
            r_last = r;
            t_last = t;
            g_last = g;
            const float w = weight(g, __builtin_amdgcn_readfirstlane(B.run_prim[r]) == h);
            if (row < RM) B.map[wave * RM + row][lane] = w;
            else R.extra[(int64_t)(row - RM) * 64 + lane] = w;
        }
    }
    if (lane == 0) B.nmap[wave] = nmap;
    R.far = R.many || R.nrow > RM;
    R.search = R.many || R.nrow > nmap;
    R.nrow = min(R.nrow, nmap);
    __syncthreads();
    return R;
}

// does the pixel range (packed int16 pairs) touch the 4x4 sub-block at (x0, y0)?
__device__ __forceinline__ bool touches4(int xr, int yr, int x0, int y0) {
    return !(hi16(xr) < x0 || lo16(xr) > x0 + 3 || hi16(yr) < y0 || lo16(yr) > y0 + 3);
}

// Which 4x4 sub-blocks of the 8x8 block at (wx0, wy0) an entry can reach (bit
// q: sub-block q), from its mean relative to the block, conic and pixel range.
// An entry counts when its support box touches the sub-block and the
// sub-block's centre is within the conic bound of sub_block_bound (an entry
// left out has no live pixel there, so the result does not change).
__device__ __forceinline__ int sub_blocks(float2 m, float4 ex, float thr, int a, int b, int wx0, int wy0) {
    // exponents at the sub-block centres (1.5 | 5.5, 1.5 | 5.5) of the block
    const float dx0 = 1.5f - m.x, dx1 = 5.5f - m.x, dy0 = 1.5f - m.y, dy1 = 5.5f - m.y;
    const float by0 = ex.y * dy0, by1 = ex.y * dy1, cy0 = ex.z * dy0 * dy0, cy1 = ex.z * dy1 * dy1;
    const bool n0 = fmaf(dx0, fmaf(ex.x, dx0, by0), cy0) < thr, n1 = fmaf(dx1, fmaf(ex.x, dx1, by0), cy0) < thr;
    const bool n2 = fmaf(dx0, fmaf(ex.x, dx0, by1), cy1) < thr, n3 = fmaf(dx1, fmaf(ex.x, dx1, by1), cy1) < thr;
    return (!n0 && touches4(a, b, wx0, wy0) ? 1 : 0) | (!n1 && touches4(a, b, wx0 + 4, wy0) ? 2 : 0) |
           (!n2 && touches4(a, b, wx0, wy0 + 4) ? 4 : 0) | (!n3 && touches4(a, b, wx0 + 4, wy0 + 4) ? 8 : 0);
}

// The entries (bits of the result, from the ballots of every lane's
// sub_blocks) that reach this lane's row's sub-block
__device__ __forceinline__ unsigned long long row_mask(int bits, int lane) {
    const unsigned long long m0 = __ballot(bits & 1), m1 = __ballot(bits & 2), m2 = __ballot(bits & 4), m3 = __ballot(bits & 8);
    const int q = lane >> 4;
    return q == 0 ? m0 : (q == 1 ? m1 : (q == 2 ? m2 : m3));
}

// index of the lowest set bit of m; 0 when m is 0, so that a row with
// nothing left reads the first entry of the half batch (always a staged,
// finite record, which its lanes then ignore)
__device__ __forceinline__ int low_bit(unsigned m) { return m ? __builtin_ctz(m) : 0; }

// do all 16 lanes of this lane's row have the flag set?
__device__ __forceinline__ bool row_all(bool f, int lane) {
    return ((__builtin_amdgcn_ballot_w64(f) >> (lane & 48)) & 0xFFFFull) == 0xFFFFull;
}



// Records of one batch slot, fetched from global memory one batch ahead of
// their use by the loader threads (tid < KI); the list entry is fetched one
// batch earlier still, so neither load stalls the wave that issues it.
struct SlotPrefetch {
    float4 r0, r1, r2, r3;
    int gp = -1;       // pixel (record index) of the records in flight
    int gp_next = -1;  // list entry for the batch after them
    __device__ __forceinline__ void load(const StatePtrs &st, int rec) {
        gp = rec;
        if (gp >= 0) {
            const float4 *rp = st.rec + (int64_t)gp * 4;
            r0 = rp[0]; r1 = rp[1]; r2 = rp[2]; r3 = rp[3];
        }
    }
    __device__ __forceinline__ void issue(const StatePtrs &st, int gs0, int n, int base_next, int tid, int K) {
        load(st, gp_next);
        const int i2 = base_next + K + tid;
        gp_next = (tid < K && i2 < n) ? (int)st.g_list[gs0 + i2] : -1;
    }
};

// For pixels q within rho of a point p, the triangle inequality in the conic's
// norm gives |q - mu|_Q >= |p - mu|_Q - sqrt(lambda_max(Q)) rho.  So no pixel
// of a 4x4 sub-block (its centres within rho = 1.5 sqrt 2 of the block's
// centre) has d^T Q d <= kappa^2 when the centre's exponent is below
// kE (kappa + sqrt(lambda_max) rho)^2; the bound is widened by 1e-3 (relative
// and absolute) so that FP32 rounding of either side never drops a live pixel.
__device__ __forceinline__ float sub_block_bound(float qa, float qb, float qc, float kappa) {
    const float h = 0.5f * (qa - qc);
    const float lmax = 0.5f * (qa + qc) + sqrtf(h * h + qb * qb);
    const float rad = (kappa + sqrtf(fmaxf(lmax, 0.0f)) * 2.1214f) * 1.001f + 1e-3f;
    return kE * rad * rad;
}

// Stages a loaded record as entry kk of the batch of wave `wave`, whose block
// starts at (wx0, wy0); returns the entry's sub_blocks (none where w = 0 on the block).
template <int KI, typename BL>
__device__ __forceinline__ int stage_slot(BatchLds<KI> &S, const SlotPrefetch &P, int kk, int wx0, int wy0, const BL &B,
                                          const RowInfo &R, unsigned own, float kappa, int wave) {
    // the pixel the Gaussian's mean is stored against
    const int a = __float_as_int(P.r2.w);
    const int x = lo16(a) - wx0, y = hi16(a) - wy0;
    const float4 ex = make_float4(kE * P.r0.z, 2.0f * kE * P.r0.w, kE * P.r1.x, P.r2.x);
    const float thr = sub_block_bound(P.r0.z, P.r0.w, P.r1.x, kappa);
    S.e[kk] = ex;
    S.c[kk] = make_float4(P.r1.y, P.r1.z, P.r1.w, 0.0f);
    const float2 m = make_float2((float)x + P.r0.x, (float)y + P.r0.y);
    const int bits = sub_blocks(m, ex, thr, __float_as_int(P.r3.x), __float_as_int(P.r3.y), wx0, wy0);
    const int g = __float_as_int(P.r2.y);
    const int r = find_run(B.run_prim, R.n_runs, g);
    int row = R.many && g > B.run_prim[BL::NR - 1] ? kSearch : kNoRow;
    if (r >= 0) {
        if constexpr (BL::NW == 1) {
            row = r < R.nrow ? r : kSearch;
        } else {
            row = (int)B.row_of[wave][r];
            row = row == 255 ? kNoRow : (row < B.nmap[wave] ? row : kSearch);
        }
    }
    S.mp[kk].m = m;
    S.mp[kk].pr = make_int2(g, row);
    return bits & (row != kNoRow ? -1 : __builtin_amdgcn_sbfe((int)own, g, 1));  // (bit g mod 32, as 0 or -1)
}

// Between a wave's writes and reads of its own batch (its LDS accesses
// complete in order: the fence keeps the compiler from moving them across each other).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------ forward

template <int TS, int K>
__global__ void __launch_bounds__(TS *TS) k_blend_fwd(Consts k, ViewTable vt, StatePtrs st, RowPool pool, float *image) {
    using G = TileGeom<TS>;
    using D = BlendDims<TS, K>;
    using BL = BoundaryLds<TS, K, D::RM_FWD>;
    constexpr int RM = BL::RM, NW = D::NW, KI = D::KI_FWD;
    __shared__ BL B;
    __shared__ BatchLds<KI> SB[NW];
    const int t = st.order[blockIdx.x], tid = threadIdx.x, lane = tid & 63;
    const int wave = NW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    BatchLds<KI> &S = SB[wave];
    const int v = view_of_tile(vt, t);
    const ViewInfo vi = vt.v[v];
    const int tl = t - vi.tile_off, tx = tl % vi.tiles_x, ty = tl / vi.tiles_x;
    int lx, ly;
    G::local_xy(tid, lx, ly);
    const int px = tx * TS + lx, py = ty * TS + ly;
    const bool inside = px < vi.W && py < vi.H;
    const int pix = vi.px_off + py * vi.W + px;
    int h = -1;
    if (inside) {
        const int tri = st.I_tri[pix];
        h = tri < 0 ? -1 : tri / k.L2;
    }
    const int ox = tx * TS, oy = ty * TS;
    const float qx = (float)(lx & 7), qy = (float)(ly & 7);  // position in the wave's 8x8 block
    const int wx0 = tx * TS + (wave % G::SPR) * 8, wy0 = ty * TS + (wave / G::SPR) * 8;

    const int bs0 = st.b_start[t], bc = st.b_count[t];
    if (bc > D::CAP && tid == 0) atomicAdd((unsigned long long *)&st.counters[C_BIGBLIST], 1ull);
    if (st.g_count[t] == 0) {
        // no Gaussian reaches the tile (most of the background): T = 1
        if (inside) {
            image[3 * (int64_t)pix + 0] = k.bg[0];
            image[3 * (int64_t)pix + 1] = k.bg[1];
            image[3 * (int64_t)pix + 2] = k.bg[2];
            st.T_final[pix] = 1.0f;
            st.last[pix] = 0;
        }
        return;
    }
    // the first batch's records are read before the boundary points are
    // staged, so that the two waits overlap
    const int gs0 = st.g_start[t], gc = st.g_count[t];
    SlotPrefetch pf;
    pf.gp_next = (lane < KI && lane < gc) ? (int)st.g_list[gs0 + lane] : -1;
    pf.issue(st, gs0, gc, 0, lane, KI);
    const RowInfo R = build_rows<TS, K, false>(B, st, pool, bs0, bc, ox, oy, lx, ly, h);
    // (a tile counts once, by the first of its waves whose runs do not fit)
    if (R.far && lane == 0 && (NW == 1 || atomicExch(&B.ws[NW], 1) == 0))
        atomicAdd((unsigned long long *)&st.counters[C_MANYRUNS], 1ull);
    const float *const map = &B.map[wave * RM][lane];

    float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
    bool done = !inside;
    int last = gc;
    const float amax = k.alpha_max, tmin = k.t_min;
    const bool nob = (k.flags & BGT_FLAG_NO_BOUNDARY) != 0;
    const unsigned own_m = nob ? ~0u : own_prims(h);
    const bool far = R.far;  // only then do the loops below look for entries without an LDS row
    // support test d^T Q d <= 2 ln(1/g_min) as a base-2 exponent: G = 2^e, e >= log2(g_min)
    const float e_min = kE * k.kappa2;
    const float kappa = sqrtf(k.kappa2);
    unsigned long long staged = 0;  // the staged batch's entries for this lane's row
    auto stage = [&] {
        int bits = 0;
        if (pf.gp >= 0) bits = stage_slot(S, pf, lane, wx0, wy0, B, R, own_m, kappa, wave);
        staged = row_mask(bits, lane);
    };
    stage();
    for (int base = 0; base < gc; base += KI) {
        wave_sync();
        if (all_lanes(done)) break;
        int stop_kk = -1;  // batch index of the entry at which this pixel stops in this batch
        pf.issue(st, gs0, gc, base + KI, lane, KI);   // next batch's records, in flight during compositing
        unsigned long long mine = staged;
        if (row_all(done, lane)) mine = 0;  // this row has stopped
#pragma unroll
        for (int hb = 0; hb < (KI > 32 ? 64 : 32); hb += 32) {
            unsigned mm = (unsigned)(mine >> hb);
            if (any_lane(mm != 0u)) do {
                // each row composites its own next entry: branch-free per
                // lane, a lane that does not composite it takes alpha = 0,
                // which leaves T and C bit-identical
                const bool act = mm != 0u;
                const int kk = hb + low_bit(mm);
                mm &= mm - 1u;
                const int2 pr = S.mp[kk].pr;
                const float2 m = S.mp[kk].m;
                const float4 ex = S.e[kk];
                const float4 c = S.c[kk];
                const int g = pr.x, r = pr.y;  // uniform within the row
                const bool own = g == h || nob;  // w = 1 for all without coefficients
                const float dx = qx - m.x, dy = qy - m.y;
                const float e = fmaf(dx, fmaf(ex.x, dx, ex.y * dy), ex.z * dy * dy);
                // w = 0 without a boundary point of g near this block, or outside the support
                bool live = act && !done && (own || r != kNoRow) && e >= e_min;
                // (at 16 and 32 px a step in which no lane's support
                // is reached leaves before the weights; T and C would
                // not change)
                if (TS >= 16 && !any_lane(live)) continue;
                // w = 0 (gamma* = 1 for another patch's Gaussian) gives
                // a = 0 with no test: T and C stay as they are
                float w = map[min(max(r, 0), RM - 1) * 64];
                w = (unsigned)r < (unsigned)RM ? w : 1.0f;
                if (far && any_lane(live && (r >= RM || r == kSearch))) {
                    if (live && r >= RM) {
                        w = R.extra[(int64_t)(r - RM) * 64 + lane];
                    } else if (live && r == kSearch) {
                        float gam;
                        search_prim(B, st, bs0, bc, g, R.n_runs, lx, ly, ox, oy, &gam);
                        w = weight(gam, own);
                    }
                }
                // min(raw, alpha_max) as integers: the same as fminf for
                // every non-NaN raw, alpha_max being positive (one
                // instruction; fminf also canonicalizes alpha_max)
                float a = __int_as_float(min(__float_as_int(ex.w * w * support_exp2(e)), __float_as_int(amax)));
                a = live ? a : 0.0f;
                const float ta = T * a;
                C0 += ta * c.x;
                C1 += ta * c.y;
                C2 += ta * c.z;
                T = T * (1.0f - a);
                // (the stopping entry's batch index; the list index is
                // formed once per batch below)
                const bool stop = live && T < tmin;
                done = done || stop;
                stop_kk = stop ? kk : stop_kk;
            } while (any_lane(mm != 0u));
        }
        if (stop_kk >= 0) last = base + stop_kk + 1;
        wave_sync();
        stage();
    }
    if (inside) {
        image[3 * (int64_t)pix + 0] = C0 + T * k.bg[0];
        image[3 * (int64_t)pix + 1] = C1 + T * k.bg[1];
        image[3 * (int64_t)pix + 2] = C2 + T * k.bg[2];
        st.T_final[pix] = T;
        st.last[pix] = last;
    }
}

// ------------------------------------------------------------ backward

// 4x4 transpose across the four rows of the wave: lane i of row j starts with
// a[s] = value of step s at its own pixel and ends with a[p] = value of step j
// at pixel i of row p.  (v_permlane16_swap exchanges the odd rows of its first
// operand with the even rows of its second, v_permlane32_swap the upper half
// of the first with the lower half of the second.)
__device__ __forceinline__ void swap16(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap32(float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void row_transpose(float (&a)[4]) {
    swap16(a[0], a[1]);
    swap16(a[2], a[3]);
    swap32(a[0], a[2]);
    swap32(a[1], a[3]);
}

// Row reduce-scatter of nine per-lane values: butterflies over lane bits 0
// (quad_perm [1,0,3,2]), 1 (quad_perm [2,3,0,1]) and 3 (row_ror:8) each halve
// the set of values a lane carries (v[0..7]; v[8] is summed in every lane),
// then row_shr:4 folds bit 2.  Afterwards, in every 16-lane row, the lane
// with bit 2 set and bits (b3, b1, b0) holds the row total of
// v[4 b3 + 2 b1 + b0] in v[0], and every lane with bit 2 set the row total
// of v[8] in v[8]: 26 VALU operations instead of 36 for nine plain row sums.
__device__ __forceinline__ void row_reduce_scatter9(float *v, int lane) {
    const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0, b3 = (lane & 8) != 0;
    float u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float keep = b0 ? v[2 * k + 1] : v[2 * k], send = b0 ? v[2 * k] : v[2 * k + 1];
        u[k] = keep + dpp_f<0xB1, 0xF>(send);
    }
    float s8 = v[8] + dpp_f<0xB1, 0xF>(v[8]);
    float w[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const float keep = b1 ? u[2 * m + 1] : u[2 * m], send = b1 ? u[2 * m] : u[2 * m + 1];
        w[m] = keep + dpp_f<0x4E, 0xF>(send);
    }
    s8 += dpp_f<0x4E, 0xF>(s8);
    const float keep = b3 ? w[1] : w[0], send = b3 ? w[0] : w[1];
    float x = keep + dpp_f<0x128, 0xF>(send);
    s8 += dpp_f<0x128, 0xF>(s8);
    x += dpp_f<0x114, 0xF>(x);  // row_shr:4
    s8 += dpp_f<0x114, 0xF>(s8);
    v[0] = x;
    v[8] = s8;
}

// Adds the boundary terms of one pixel for dl/dgamma* = dg to the point of
// record bpix, at tile pixel (lx, ly): add(which, value), which = 0 sigma,
// 1 and 2 the position.
template <typename Add>
__device__ __forceinline__ void route_boundary(const StatePtrs &st, int bpix, float dg, int lx, int ly, int ox, int oy,
                                               Add &&add) {
    constexpr float LN2 = 0.69314718055994531f;
    const float4 r0 = st.rec[(int64_t)bpix * 4];
    const float4 r2 = st.rec[(int64_t)bpix * 4 + 2];
    const int a = __float_as_int(r2.w);
    const float dx = (float)(lx - (lo16(a) - ox)) - r0.x, dy = (float)(ly - (hi16(a) - oy)) - r0.y;
    const float sg = r2.z, d = bdist(dx, dy);
    const float gam = gamma_fn(d, sg);  // gamma of the routed point (gamma* up to FP32 rounding)
    const float dd = dg * LN2 / sg * gam;
    if (d > kDKink) {
        add(1, -dd * dx / d);
        add(2, -dd * dy / d);
    }
    add(0, -dg * LN2 * d / (sg * sg) * gam);
}

// Front-to-back replay of the forward per pixel: T_i is recomputed exactly as
// the forward did, the suffix S_i = sum_{j>i} T_j a_j c_j + T_n bg is the
// forward colour minus the running prefix (carried as its dot product with
// dl/dC), and
//   dl/dc_i = T_i a_i dl/dC,  dl/da_i = dl/dC . (T_i c_i - S_i / (1 - a_i)),
//   dl/dw = dl/da a / w (Supplementary Sec. C), G = exp(-d^T Q d / 2).
// The wave walks the entries that reach its block four at a time, every lane
// its own pixel.  (Rows walking their own entries, as in the forward, take as
// many steps: entries in depth order come in clusters that one or two of the
// four sub-blocks hold, 13.9 M row steps for 14.3 M entries.)  An entry leaves
// two scalars per pixel, dl/do and T a; every sum it needs is linear in one of
// them with factors that depend on the pixel alone (its offset, dl/dC).  So
// the four entries' scalars are transposed across the wave's rows: a lane then
// has its row's entry at four pixels (4 px apart), forms the nine sums over
// them (the moments from sums at x and y offsets 0 and 4, shifted to the
// entry's mean), and one row reduce-scatter finishes four entries at once.
// What bounds the kernel is VALU issue: reducing nine products per pixel and
// entry over the whole wave took 36 of 90 VALU instructions per entry, this
// takes 18.  At 8 px the totals are the tile's and go to the records' slots for
// the tile (plain stores: the parameter pass sums a record's slots over its
// tiles in a fixed order, so the result does not depend on scheduling; a
// record reaching more than 3 x 3 tiles adds into sums of its own by float
// atomics instead); larger tiles add their waves' totals in LDS first, in a
// ring of batches, each stored by the last wave to finish it: with a barrier
// per 64 entries the waves waited for the slowest a third of the time (four
// views of 800x800, 16 px tiles: 0.92 -> 0.78 ms, 32 px 2.6 -> 2.2 ms; 0.69 and 1.57
// now).
// The boundary terms accumulate per (row, pixel), as the sum of dl/dw, in
// registers for the LDS rows (the row is wave-uniform), and go to the
// minimising boundary point at the end.  16 views of 800x800, 2000 patches, 8 px
// tiles: 2.25 -> 1.80 ms, 1.43e9 -> 0.94e9 VALU instructions (1.73 ms now); 50,000
// patches at 32 x 1024x768: 7.35 -> 4.11 ms (with the rows above; 3.80 now); 8000
// cubic patches at 1000x1000, 16 px tiles: 3.39 -> 0.43 ms (rows per 8x8 block;
// 0.34 now).
// Waves per SIMD the registers must allow.
template <int TS, int K>
struct BwdWaves {
    static constexpr int value = TS == 32 ? 1 : 5;
};

template <int TS, int K>
__global__ void __launch_bounds__(TS *TS) __attribute__((amdgpu_waves_per_eu(BwdWaves<TS, K>::value)))
k_blend_bwd(Consts k, ViewTable vt, StatePtrs st, RowPool pool, const float *image, const float *grad_image) {
    using G = TileGeom<TS>;
    using D = BlendDims<TS, K>;
    using BL = BoundaryLds<TS, K, D::RM_BWD>;
    constexpr int RM = BL::RM, NW = D::NW, KI = D::KI_BWD, CAP = D::CAP;
    constexpr bool ONE = NW == 1;
    __shared__ BL B;
    // sums of dl/dw per LDS row at this pixel (uniform index: indexed
    // registers; with fewer than about ten entries the compiler would index
    // the array by select chains)
    constexpr int RD = RM < 12 ? 12 : RM;
    float dgr[RD];
#pragma unroll
    for (int i = 0; i < RD; ++i) dgr[i] = 0.f;
    // the batch and its sums are dead once the list is done; the per-point
    // boundary sums reuse their space
    // larger tiles: batches of the list whose sums the waves add up in LDS
    constexpr int RING = ONE ? 1 : 4;
    struct LoopLds {
        BatchLds<KI> S[NW];
        float acc[ONE ? 1 : RING * KI * kSums];
    };
    union TailLds {
        LoopLds loop;
        float bacc[CAP][3];
    };
    __shared__ TailLds U;
    __shared__ int max_last;
    __shared__ int ring_done[RING], ring_free[RING];  // waves that finished a slot's batches; batches stored from it
    float *acc = U.loop.acc;  // (the batch's first entry's sums)
    const int t = st.order[blockIdx.x], tid = threadIdx.x, lane = tid & 63;
    const int wave = NW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    BatchLds<KI> &S = U.loop.S[wave];
    const int gc = st.g_count[t];
    if (gc == 0) {  // no Gaussian reaches the tile: nothing to differentiate
        if (tid == 0) st.t_end[t] = 0;
        return;
    }
    const int v = view_of_tile(vt, t);
    const ViewInfo vi = vt.v[v];
    const int tl = t - vi.tile_off, tx = tl % vi.tiles_x, ty = tl / vi.tiles_x;
    int lx, ly;
    G::local_xy(tid, lx, ly);
    const int px = tx * TS + lx, py = ty * TS + ly;
    const bool inside = px < vi.W && py < vi.H;
    const int pix = vi.px_off + py * vi.W + px;
    int h = -1, mylast = 0;
    float g0 = 0.f, g1 = 0.f, g2 = 0.f, im0 = 0.f, im1 = 0.f, im2 = 0.f;
    if (inside) {
        const int tri = st.I_tri[pix];
        h = tri < 0 ? -1 : tri / k.L2;
        mylast = min(max(st.last[pix], 0), gc);
        g0 = grad_image[3 * (int64_t)pix]; g1 = grad_image[3 * (int64_t)pix + 1]; g2 = grad_image[3 * (int64_t)pix + 2];
        im0 = image[3 * (int64_t)pix]; im1 = image[3 * (int64_t)pix + 1]; im2 = image[3 * (int64_t)pix + 2];
        if (g0 == 0.f && g1 == 0.f && g2 == 0.f) mylast = 0;
    }
    const int ox = tx * TS, oy = ty * TS;
    const float qx = (float)(lx & 7), qy = (float)(ly & 7);
    const int wx0 = tx * TS + (wave % G::SPR) * 8, wy0 = ty * TS + (wave / G::SPR) * 8;
    // this tile's slot of the narrow records' sums
    float *const gs_tile = st.gslot + (int64_t)tile_slot(tx, ty) * st.n_rec * kSums;

    int wave_last = mylast;  // last list entry any lane of this wave (the tile) replays
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) wave_last = max(wave_last, __shfl_xor(wave_last, o, 64));
    wave_last = __builtin_amdgcn_readfirstlane(wave_last);
    int nlast = wave_last;

    // the first batch's records are read before the boundary points are
    // staged, so that the two waits overlap (entries past the replayed
    // prefix, known once the stop indices are combined, are dropped then)
    const int gs0 = st.g_start[t];
    SlotPrefetch P;
    P.load(st, (lane < KI && lane < gc) ? (int)st.g_list[gs0 + lane] : -1);
    const int bs0 = st.b_start[t], bc = st.b_count[t];
    if constexpr (NW > 1) {
        if (tid == 0) max_last = 0;
        if (tid < RING) ring_done[tid] = ring_free[tid] = 0;
        __syncthreads();
        if (lane == 0) atomicMax(&max_last, wave_last);
    }
    if constexpr (!ONE)
        for (int i = tid; i < RING * KI * kSums; i += TS * TS) acc[i] = 0.f;
    const RowInfo R = build_rows<TS, K, true>(B, st, pool, bs0, bc, ox, oy, lx, ly, h);  // (syncs)
    if constexpr (NW > 1) nlast = max_last;
    const float *const map = &B.map[wave * RM][lane];
    // (the extra gamma* rows, then as many of dl/dw)
    float *const dextra = R.extra ? R.extra + (int64_t)(R.nrow - RM) * 64 + lane : nullptr;

    if (tid == 0) st.t_end[t] = gs0 + nlast;  // the prefix of the list whose sums are written below
    // dl/dC . S: the suffix colour S = C - prefix enters dl/dalpha only through
    // its dot product with dl/dC, so that product is carried instead of S
    float T = 1.0f, GS = g0 * im0 + g1 * im1 + g2 * im2;
    const float amax = k.alpha_max;
    const bool nob = (k.flags & BGT_FLAG_NO_BOUNDARY) != 0;
    const LaneMask nob_m = nob ? ~0ull : 0ull;
    const unsigned own_m = nob ? ~0u : own_prims(h);
    const float e_min = kE * k.kappa2;
    const float kappa = sqrtf(k.kappa2);
    // pixel i of this lane's row's sub-block in each of the four: its place in
    // the first and dl/dC there
    const float bx = (float)(lane & 3), by = (float)((lane >> 2) & 3);
    float gq[3][4];
    {
        const float gv[3] = {g0, g1, g2};
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int p = 0; p < 4; ++p) gq[c][p] = __shfl(gv[c], p * 16 + (lane & 15), 64);
    }

    // Takes the next entry of the mask that any lane's support reaches (kk,
    // wave-uniform; -1: none left) and replays it at this lane's pixel if it is
    // one of the first `left` of the batch: leaves dl/do and T a.  SEARCH:
    // entries may need the per-pixel search
    auto replay = [&](unsigned long long &mask, int left, float &d_o, float &ta, auto search) -> int {
        constexpr bool SEARCH = decltype(search)::value;
        int kk = -1, g = 0, r = 0;
        float4 ex = make_float4(0.f, 0.f, 0.f, 0.f);
        float e = 0.f;
        LaneMask live_m = 0ull;
        d_o = 0.f;
        ta = 0.f;
        while (true) {
            if (!mask) return -1;
            kk = __ffsll((long long)mask) - 1;
            mask &= mask - 1;
            const int2 prk = S.mp[kk].pr;
            const float2 m = S.mp[kk].m;
            ex = S.e[kk];
            g = prk.x;
            r = __builtin_amdgcn_readfirstlane(prk.y);
            const float dx = qx - m.x, dy = qy - m.y;
            e = fmaf(dx, fmaf(ex.x, dx, ex.y * dy), ex.z * dy * dy);  // as in the forward
            live_m = lanes(kk < left) & lanes(e >= e_min);
            if (r == kNoRow) live_m &= lanes(g == h) | nob_m;  // w = 1 on its own pixels (all without coefficients), else 0
            if (live_m) break;
        }
        const bool live = in_mask(live_m);
        const float4 c = S.c[kk];
        float w = 1.0f;
        int arg = -1;
        if (r >= 0) {
            if (r < RM) w = map[r * 64];
            else w = R.extra[(int64_t)(r - RM) * 64 + lane];
        }
        if constexpr (SEARCH)
            if (r == kSearch && live) {
                float gam;
                arg = search_prim(B, st, bs0, bc, g, R.n_runs, lx, ly, ox, oy, &gam);
                w = weight(gam, g == h);
            }
        const float Gv = support_exp2(e);
        const float raw = ex.w * w * Gv;
        const bool smooth = in_mask(live_m & ~lanes(raw > amax));
        // min(raw, alpha_max) as integers, as in the forward (the same as the
        // clamp for every non-NaN raw, alpha_max being positive)
        float a = __int_as_float(min(__float_as_int(raw), __float_as_int(amax)));
        a = live ? a : 0.0f;
        ta = T * a;
        const float gcol = g0 * c.x + g1 * c.y + g2 * c.z;  // dl/dC . c_i
        GS -= ta * gcol;
        const float inv = __builtin_amdgcn_rcpf(1.0f - a);
        const float dalpha = T * gcol - GS * inv;
        T = T * (1.0f - a);
        const float q = smooth ? dalpha * Gv : 0.0f;
        d_o = q * w;
        // dl/dw of the run at this pixel (where gamma* = 1 the sum is dropped at
        // the end: w does not move there)
        if (r >= 0) {
            if (r < RM) dgr[r] += q * ex.w;
            else dextra[(int64_t)(r - RM) * 64] += q * ex.w;
        } else if constexpr (SEARCH) {
            if (arg >= 0 && q != 0.0f) {
                const float dw = q * ex.w;
                const int bpix = (int)st.b_list[bs0 + arg];
                route_boundary(st, bpix, g == h ? dw : -dw, lx, ly, ox, oy,
                               [&](int f, float x) { unsafeAtomicAdd(&st.dbound[(int64_t)bpix * 3 + f], x); });
            }
        }
        return kk;
    };
    // the sums of entries k0..k3 (d, ta: dl/do and T a of each; -1: none), row j
    // finishing entry kj
    auto add_sums = [&](int k0, int k1, int k2, int k3, float (&d)[4], float (&ta)[4]) {
        row_transpose(d);
        row_transpose(ta);
        const int j = lane >> 4;
        const int kj = j == 0 ? k0 : (j == 1 ? k1 : (j == 2 ? k2 : k3)), kq = max(kj, 0);
        const float2 m = S.mp[kq].m;
        const float o = S.e[kq].w;
        const float dx = bx - m.x, dy = by - m.y;
        const float sx = d[1] + d[3], sy = d[2] + d[3], s = sx + (d[0] + d[2]);
        // (the moments are of dl/dG G = o dl/do)
        const float o4 = 4.0f * o, so = o * s, x4 = o4 * sx, y4 = o4 * sy;
        float v[kSums];
        v[0] = fmaf(so, dx, x4);  // sum dG (dx + 4 X)
        v[1] = fmaf(so, dy, y4);  // sum dG (dy + 4 Y)
        v[2] = fmaf(dx, v[0] + x4, 4.0f * x4);
        v[3] = fmaf(dx, v[1], fmaf(dy, x4, 4.0f * o4 * d[3]));
        v[4] = fmaf(dy, v[1] + y4, 4.0f * y4);
#pragma unroll
        for (int c = 0; c < 3; ++c)
            v[5 + c] = fmaf(ta[3], gq[c][3], fmaf(ta[2], gq[c][2], fmaf(ta[1], gq[c][1], ta[0] * gq[c][0])));
        v[8] = s;
        row_reduce_scatter9(v, lane);
        if ((lane & 4) && kj >= 0) {
            const int f = ((lane >> 1) & 4) | (lane & 3);
            if constexpr (ONE) {
                const int rec = __float_as_int(S.c[kq].w);  // (~record of a wide one)
                if (rec >= 0) {
                    float *dst = gs_tile + (int64_t)rec * kSums;
                    dst[f] = v[0];
                    if ((lane & 15) == 4) dst[8] = v[8];
                } else {
                    float *dst = st.gwide + (int64_t)~rec * kSums;
                    unsafeAtomicAdd(&dst[f], v[0]);
                    if ((lane & 15) == 4) unsafeAtomicAdd(&dst[8], v[8]);
                }
            } else {
                float *dst = acc + kq * kSums;
                atomicAdd(&dst[f], v[0]);
                if ((lane & 15) == 4) atomicAdd(&dst[8], v[8]);
            }
        }
    };

    constexpr int TSH = TS == 8 ? 3 : (TS == 16 ? 4 : 5);
    int cur_gp = lane < wave_last ? P.gp : -1;
    bool wide = false;                    // this lane's entry adds to sums of its own
    unsigned long long staged = 0;        // the staged batch's entries that reach the block
    auto stage = [&](const SlotPrefetch &Q) {  // Q's record as this lane's entry; whether it reaches the block
        wide = !narrow_range(__float_as_int(Q.r3.x), __float_as_int(Q.r3.y), TSH);
        const int bits = stage_slot(S, Q, lane, wx0, wy0, B, R, own_m, kappa, wave);
        if constexpr (ONE) S.c[lane].w = __int_as_float(wide ? ~Q.gp : Q.gp);
        return bits != 0;
    };
    {
        bool reaches = false;
        if (cur_gp >= 0) reaches = stage(P);
        staged = __ballot(reaches);
    }
    for (int base = 0; base < nlast; base += KI) {
        wave_sync();
        unsigned stored = 0u;            // (8 px) entries whose sums went to memory
        const int left = mylast - base;  // entries this lane replays
        unsigned long long mask = staged;
        const int slot = base / KI % RING, gen = base / KI / RING;  // (larger tiles)
        if constexpr (!ONE) {
            // the slot's last batch has been stored
            acc = U.loop.acc + slot * KI * kSums;
            while (__hip_atomic_load(&ring_free[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < gen)
                __builtin_amdgcn_s_sleep(1);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        }
        if (R.search) {  // (rare) one entry at a time
            while (mask) {
                float d[4] = {0.f, 0.f, 0.f, 0.f}, ta[4] = {0.f, 0.f, 0.f, 0.f};
                const int kk = replay(mask, left, d[0], ta[0], std::true_type());
                if (kk < 0) break;
                if constexpr (ONE) stored |= 1u << kk;
                add_sums(kk, -1, -1, -1, d, ta);
            }
        } else {
            while (mask) {
                float d[4], ta[4];
                int ks[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    ks[s] = replay(mask, left, d[s], ta[s], std::false_type());
                    if constexpr (ONE) stored |= ks[s] >= 0 ? 1u << ks[s] : 0u;
                }
                if (ks[0] < 0) break;
                add_sums(ks[0], ks[1], ks[2], ks[3], d, ta);
            }
        }
        wave_sync();
        // the next batch is staged before this batch's sums are stored: a
        // load issued after the stores would wait for them too
        const int prev_gp = cur_gp;
        const bool prev_wide = wide;
        cur_gp = lane < KI && base + KI + lane < wave_last ? (int)st.g_list[gs0 + base + KI + lane] : -1;
        bool reaches = false;
        if (cur_gp >= 0) {
            SlotPrefetch Q;
            Q.load(st, cur_gp);
            reaches = stage(Q);
        }
        staged = __ballot(reaches);
        if constexpr (ONE) {
            // zero sums for the entries that do not reach the block
            if (lane < KI && prev_gp >= 0 && !prev_wide && !((stored >> lane) & 1u))
                zero_sums(gs_tile + (int64_t)prev_gp * kSums);
        } else {
            // the last wave to finish a batch stores and clears its sums.  A
            // wave may be up to RING batches ahead of the slowest: its wait
            // above is for a batch that every wave is past, or storing, so the
            // slowest never waits for another
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            int before = 0;
            if (lane == 0)
                before = __hip_atomic_fetch_add(&ring_done[slot], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (__builtin_amdgcn_readfirstlane(before) == NW * (gen + 1) - 1) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                int gp = prev_gp;
                bool wd = prev_wide;
                if (gp < 0 && lane < KI && base + lane < nlast) {  // (past the last entry this wave replays)
                    gp = (int)st.g_list[gs0 + base + lane];
                    const int2 range = *(const int2 *)(st.rec + (int64_t)gp * 4 + 3);
                    wd = !narrow_range(range.x, range.y, TSH);
                }
                if (gp >= 0) {
                    float *a = acc + lane * kSums;
                    if (wd) {
                        float *dst = st.gwide + (int64_t)gp * kSums;
#pragma unroll
                        for (int f = 0; f < kSums; ++f)
                            if (a[f] != 0.f) unsafeAtomicAdd(&dst[f], a[f]);
                    } else {
                        float *dst = gs_tile + (int64_t)gp * kSums;
#pragma unroll
                        for (int f = 0; f < kSums; ++f) dst[f] = a[f];
                    }
#pragma unroll
                    for (int f = 0; f < kSums; ++f) a[f] = 0.f;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                if (lane == 0)
                    __hip_atomic_store(&ring_free[slot], gen + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    // boundary points at the arg-min of each (run, pixel): d gamma / d b,
    // d sigma.  The arg-min is searched over the run (arg_min: the smallest
    // d/sigma, near-ties decided in FP64, the lowest raster index among
    // exactly equal ratios).
    __syncthreads();  // the loaders' last flush reads acc, which bacc overlays
    const int in_lds = bc <= CAP ? bc : 0;  // (a list staged in chunks is read from its records)
    float(&bacc)[CAP][3] = U.bacc;
    for (int i = tid; i < in_lds * 3; i += TS * TS) (&bacc[0][0])[i] = 0.f;
    __syncthreads();
    for (int r = 0; r < R.n_runs; ++r) {
        int row = r;
        if constexpr (NW > 1) row = __builtin_amdgcn_readfirstlane((int)B.row_of[wave][r]);
        if (row >= R.nrow) continue;  // (no row, or the run does not reach the block)
        float dg = 0.f;  // dgr[row] by selects (row is uniform; dgr stays in registers)
        if (row < RM) {
#pragma unroll
            for (int i = 0; i < RM; ++i) dg = i == row ? dgr[i] : dg;
        } else {
            dg = dextra[(int64_t)(row - RM) * 64];
        }
        const bool own = B.run_prim[r] == h;
        const float w = row < RM ? map[row * 64] : R.extra[(int64_t)(row - RM) * 64 + lane];
        if (dg == 0.f || w == (own ? 1.0f : 0.0f)) continue;  // (gamma* = 1)
        const int e = arg_min(B, st, bs0, B.run_start[r], B.run_start[r + 1], in_lds, lx, ly, ox, oy, (float *)nullptr);
        if (e < 0) continue;
        // dl/dgamma*: w = gamma* on the run's own pixels, 1 - gamma* elsewhere
        const int bpix = (int)st.b_list[bs0 + e];
        route_boundary(st, bpix, own ? dg : -dg, lx, ly, ox, oy, [&](int f, float x) {
            if (in_lds > 0) atomicAdd(&bacc[e][f], x);
            else unsafeAtomicAdd(&st.dbound[(int64_t)bpix * 3 + f], x);
        });
    }
    __syncthreads();
    for (int e = tid; e < in_lds; e += TS * TS) {
        const float a0 = bacc[e][0], a1 = bacc[e][1], a2 = bacc[e][2];
        if (a0 == 0.f && a1 == 0.f && a2 == 0.f) continue;
        float *dst = st.dbound + (int64_t)st.b_list[bs0 + e] * 3;
        if (a0 != 0.f) unsafeAtomicAdd(&dst[0], a0);
        if (a1 != 0.f) unsafeAtomicAdd(&dst[1], a1);
        if (a2 != 0.f) unsafeAtomicAdd(&dst[2], a2);
    }
}

static RowPool row_pool(const Consts &k, const StatePtrs &st, int counter) {
    RowPool p;
    p.a = (float *)st.g_keys;
    p.b = (float *)st.b_keys;
    p.na = k.cap_g * 8 / 256;
    p.nb = k.cap_b * 8 / 256;
    p.next = (unsigned long long *)&st.counters[counter];
    return p;
}

template <int TS, int K>
static hipError_t launch_fwd_t(const Consts &k, const ViewTable &vt, const StatePtrs &st, float *image, hipStream_t s) {
    hipLaunchKernelGGL((k_blend_fwd<TS, K>), dim3(vt.total_tiles), dim3(TS * TS), 0, s, k, vt, st,
                       row_pool(k, st, C_ROWS_FWD), image);
    return hipGetLastError();
}

template <int TS, int K>
static hipError_t launch_bwd_t(const Consts &k, const ViewTable &vt, const StatePtrs &st, const float *image,
                               const float *grad, hipStream_t s) {
    hipLaunchKernelGGL((k_blend_bwd<TS, K>), dim3(vt.total_tiles), dim3(TS * TS), 0, s, k, vt, st,
                       row_pool(k, st, C_ROWS_BWD), image, grad);
    return hipGetLastError();
}

// (tile, batch) pairs and the kernel they take: `batch` tells the two 8 px
// variants apart, larger tiles have one kernel
#define BGT_BLEND_CONFIGS(X) \
    X(8, 32, 32) X(8, 64, 64) X(16, 32, 64) X(16, 64, 64) X(16, 128, 64) X(32, 32, 64) X(32, 64, 64) X(32, 128, 64)

hipError_t launch_blend_fwd(const Consts &k, const ViewTable &vt, const StatePtrs &st, float *image, hipStream_t s) {
#define BGT_CASE(TS, BATCH, K) \
    if (k.tile == TS && k.batch == BATCH) return launch_fwd_t<TS, K>(k, vt, st, image, s);
    BGT_BLEND_CONFIGS(BGT_CASE)
#undef BGT_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_blend_bwd(const Consts &k, const ViewTable &vt, const StatePtrs &st, const float *image,
                            const float *grad_image, hipStream_t s) {
#define BGT_CASE(TS, BATCH, K) \
    if (k.tile == TS && k.batch == BATCH) return launch_bwd_t<TS, K>(k, vt, st, image, grad_image, s);
    BGT_BLEND_CONFIGS(BGT_CASE)
#undef BGT_CASE
    return hipErrorInvalidValue;
}

}  // namespace bgt
