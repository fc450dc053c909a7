// Tile binning for the rendering acceleration of Sec. 3.2: Gaussians go to
// every tile their support reaches, sorted front to back within the tile;
// boundary points go to every tile their radius reaches, sorted by primitive
// id.  The sort is a two-level radix split: a counting pass on the tile id
// (the high key digit) places each pair in its tile's segment, then each
// segment is sorted on the low digits (depth, record index) or (primitive,
// record index): by one wave in registers (a bitonic network over up to 512
// keys), longer segments by a workgroup (see k_sort_long).  The low digits
// make every key unique, so the result does not depend on the order of the
// atomics that filled the segment.
#include "bgt_internal.h"

namespace bgt {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kScanBlock = kScanThreads * kScanItems;  // 1024

// inclusive scan over a wave (64 lanes)
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
    const int lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    return x;
}

// exclusive block scan of one value per thread; returns the block total
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T x, T &total, T *lds_waves) {
    const int lane = __lane_id(), wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    T inc = wave_inclusive_scan(x);
    if (lane == 63) lds_waves[wave] = inc;
    __syncthreads();
    if (wave == 0) {
        T w = lane < nw ? lds_waves[lane] : T(0);
        T wi = wave_inclusive_scan(w);
        if (lane < nw) lds_waves[lane] = wi - w;
        if (lane == nw - 1) lds_waves[32] = wi;
    }
    __syncthreads();
    T res = inc - x + lds_waves[wave];
    total = lds_waves[32];
    __syncthreads();
    return res;
}

// The blend passes take the tiles with the longest Gaussian lists first: a
// tile's time is proportional to its list, and a long one that starts last
// leaves the chip waiting for it; a view's few hundred long lists also spread
// evenly over the SIMDs.  (Backward and forward in ms, raster order -> this one:
// 2000 patches in 16 views of 800x800, 8 px tiles, 1.80 -> 1.73 and 0.775 -> 0.751,
// their lattice at 16 px 2.02 -> 1.84 and 0.93 -> 0.84; 50,000 patches in 32 views of
// 1024x768 3.97 -> 3.80 and 2.03 -> 1.91; one view of 800x800 0.214 -> 0.187 and 0.104
// -> 0.084.  Giving each XCD runs of 64 consecutive places makes no difference: 1.727
// and 1.727.  The order costs 2 us in the scan, 7 at 393000 tiles.)  Classes are an
// eighth of an octave wide (in raster order within one, roughly), the longest class
// 0, empty lists last.
__device__ __forceinline__ int order_class(int len) {
    if (len < 8) return kOrderClasses - 1 - len;
    const int e = 31 - __clz(len);  // >= 3
    return kOrderClasses - 1 - (8 * (e - 2) + ((len >> (e - 3)) & 7));
}

// Counts a tile with `len` entries (`in`: there is a tile) in the workgroup's
// classes; returns its rank in its class.  A wave's empty tiles are counted
// together.  Called by whole waves.
__device__ __forceinline__ int order_count(int *classes, bool in, int len) {
    const int lane = __lane_id();
    const unsigned long long empty = __ballot(in && len == 0);
    int first = 0;
    if (empty && lane == __ffsll((long long)empty) - 1) first = atomicAdd(&classes[kOrderClasses - 1], __popcll(empty));
    if (empty) first = __builtin_amdgcn_readlane(first, __ffsll((long long)empty) - 1);
    int rank = first + __popcll(empty & ((1ull << lane) - 1ull));
    if (in && len != 0) rank = atomicAdd(&classes[order_class(len)], 1);
    return rank;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_reduce(const int32_t *gc, const int32_t *bc, int n,
                                                              int64_t *sums, int nb, int32_t *classes) {
    __shared__ int64_t ws[33];
    __shared__ int own[kOrderClasses];
    static_assert(kScanThreads == kOrderClasses, "one class per thread");
    own[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * kScanBlock + threadIdx.x * kScanItems;
    int64_t sg = 0, sb = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i)
    {
        const bool in = base + i < n;
        const int g = in ? gc[base + i] : 0;
        sg += g;
        if (in) sb += bc[base + i];
        order_count(own, in, g);
    }
    int64_t tg, tb;
    block_exclusive_scan<int64_t>(sg, tg, ws);
    block_exclusive_scan<int64_t>(sb, tb, ws);
    if (threadIdx.x == 0) { sums[blockIdx.x] = tg; sums[nb + blockIdx.x] = tb; }
    if (own[threadIdx.x]) atomicAdd(&classes[threadIdx.x], own[threadIdx.x]);  // (the scans above are barriers)
}

// exclusive scan of the block sums (one block), totals into the counters; the
// tiles per class become the classes' first places in the order
__global__ void __launch_bounds__(1024) k_scan_top(int64_t *sums, int nb, int64_t *counters, int32_t *classes) {
    __shared__ int64_t ws[33];
    {
        const int c = threadIdx.x;
        int64_t tot;
        const int64_t ex = block_exclusive_scan<int64_t>(c < kOrderClasses ? classes[c] : 0, tot, ws);
        if (c < kOrderClasses) classes[c] = (int32_t)ex;
    }
    for (int which = 0; which < 2; ++which) {
        int64_t carry = 0;
        int64_t *s = sums + (int64_t)which * nb;
        for (int base = 0; base < nb; base += blockDim.x) {
            const int i = base + threadIdx.x;
            int64_t x = i < nb ? s[i] : 0, tot;
            int64_t ex = block_exclusive_scan<int64_t>(x, tot, ws);
            if (i < nb) s[i] = ex + carry;
            carry += tot;
        }
        if (threadIdx.x == 0) counters[which == 0 ? C_GPAIRS : C_BPAIRS] = carry;
    }
}

// The segments of a thread's kScanItems consecutive tiles from `base`, whose
// first starts at `off`: starts, cursors, and counts cut at the capacity.
// Returns whether any was cut.
__device__ __forceinline__ bool scan_write(int32_t *cnt, int32_t *st, int32_t *cur, int base, int n, int64_t off,
                                           const int32_t *v, int64_t cap) {
    bool ovf = false;
    int32_t c4[kScanItems], s4[kScanItems];
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
        int64_t c = v[i];
        if (off + c > cap) { c = off < cap ? cap - off : 0; ovf |= base + i < n; }
        s4[i] = (int32_t)(off < cap ? off : cap);
        c4[i] = (int32_t)c;
        off += v[i];
    }
    static_assert(kScanItems == 4, "one 16-byte store each");
    if (base + kScanItems <= n) {  // (base is a multiple of 4, the arrays start on 256 bytes)
        *(int4 *)(st + base) = *(int4 *)(cur + base) = make_int4(s4[0], s4[1], s4[2], s4[3]);
        if (ovf) *(int4 *)(cnt + base) = make_int4(c4[0], c4[1], c4[2], c4[3]);
    } else {
#pragma unroll
        for (int i = 0; i < kScanItems; ++i)
            if (base + i < n) { st[base + i] = cur[base + i] = s4[i]; cnt[base + i] = c4[i]; }
    }
    return ovf;
}

// a thread's kScanItems consecutive counts from `base` (0 past the end)
__device__ __forceinline__ void scan_read(const int32_t *cnt, int base, int n, int32_t *v) {
    if (base + kScanItems <= n) {
        const int4 q = *(const int4 *)(cnt + base);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) v[i] = base + i < n ? cnt[base + i] : 0;
    }
}

__global__ void __launch_bounds__(kScanThreads) k_scan_down(int32_t *gc, int32_t *gs, int32_t *gcur, int32_t *bc,
                                                            int32_t *bs, int32_t *bcur, const int64_t *sums,
                                                            int n, int nb, int64_t cap_g, int64_t cap_b,
                                                            int64_t *counters, int32_t *classes, int32_t *order) {
    __shared__ int64_t ws[33];
    __shared__ int own[kOrderClasses];
    own[threadIdx.x] = 0;
    __syncthreads();
    const int base = blockIdx.x * kScanBlock + threadIdx.x * kScanItems;
    for (int which = 0; which < 2; ++which) {
        int32_t *cnt = which == 0 ? gc : bc;
        int32_t v[kScanItems];
        scan_read(cnt, base, n, v);
        if (which == 0) {  // the tiles' places in the order
            int rank[kScanItems];
#pragma unroll
            for (int i = 0; i < kScanItems; ++i) rank[i] = order_count(own, base + i < n, v[i]);
            __syncthreads();
            const int mine = own[threadIdx.x];
            __syncthreads();
            if (mine) own[threadIdx.x] = atomicAdd(&classes[threadIdx.x], mine);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kScanItems; ++i)
                if (base + i < n) order[own[order_class(v[i])] + rank[i]] = base + i;
        }
        int64_t s = 0, tot;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) s += v[i];
        const int64_t off = block_exclusive_scan<int64_t>(s, tot, ws) + sums[(int64_t)which * nb + blockIdx.x];
        if (scan_write(cnt, which == 0 ? gs : bs, which == 0 ? gcur : bcur, base, n, off, v, which == 0 ? cap_g : cap_b))
            atomicOr((unsigned long long *)&counters[C_OVERFLOW], which == 0 ? 1ull : 2ull);
    }
}

// The tile order and the whole scan in one launch of three workgroups of 1024
// threads, for up to kScanOne tiles: the order, the Gaussian lists and the
// boundary lists.  All counts are loaded at once, four per thread in each of
// four rounds of 4096 tiles, whose scans then follow each other.  10000
// tiles: 9 us, where the other path's three launches take 19 and two gaps.
constexpr int kScanRounds = 4, kScanOne = 1024 * kScanItems * kScanRounds;
constexpr int kOrderFrom = 1024;  // fewer tiles are on the chip at once, in whatever order

__global__ void __launch_bounds__(1024) k_scan_one(int32_t *gc, int32_t *gs, int32_t *gcur, int32_t *bc, int32_t *bs,
                                                   int32_t *bcur, int n, int64_t cap_g, int64_t cap_b,
                                                   int64_t *counters, int32_t *order) {
    __shared__ int64_t ws[33];
    const bool g = blockIdx.x != 2;  // (0: order, 1: Gaussian lists, 2: boundary lists)
    int32_t *cnt = g ? gc : bc;
    int32_t v[kScanRounds][kScanItems];
#pragma unroll
    for (int r = 0; r < kScanRounds; ++r) scan_read(cnt, (r * 1024 + threadIdx.x) * kScanItems, n, v[r]);
    if (blockIdx.x == 0) {
        // (the counts may be cut at the capacity by the next workgroup
        // meanwhile: each is read once, so the places are a permutation all the same)
        __shared__ int own[kOrderClasses];
        __shared__ uint16_t place[kScanOne];  // the order, put together here and stored in runs
        if (n <= kOrderFrom) {
            if ((int)threadIdx.x < n) order[threadIdx.x] = threadIdx.x;
            return;
        }
        int rank[kScanRounds][kScanItems];
        if (threadIdx.x < kOrderClasses) own[threadIdx.x] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r)
            if (r * 1024 * kScanItems < n)
#pragma unroll
                for (int i = 0; i < kScanItems; ++i)
                    rank[r][i] = order_count(own, (r * 1024 + (int)threadIdx.x) * kScanItems + i < n, v[r][i]);
        __syncthreads();
        int64_t tot;
        const int64_t ex = block_exclusive_scan<int64_t>(threadIdx.x < kOrderClasses ? own[threadIdx.x] : 0, tot, ws);
        if (threadIdx.x < kOrderClasses) own[threadIdx.x] = (int)ex;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kScanRounds; ++r)
#pragma unroll
            for (int i = 0; i < kScanItems; ++i) {
                const int t = (r * 1024 + (int)threadIdx.x) * kScanItems + i;
                if (t < n) place[own[order_class(v[r][i])] + rank[r][i]] = (uint16_t)t;
            }
        __syncthreads();
        for (int i = threadIdx.x; i < n; i += 1024) order[i] = place[i];
        return;
    }
    int64_t carry = 0;
    bool ovf = false;
#pragma unroll
    for (int r = 0; r < kScanRounds; ++r) {
        if (r * 1024 * kScanItems >= n) break;
        int64_t s = 0, tot;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) s += v[r][i];
        const int64_t off = block_exclusive_scan<int64_t>(s, tot, ws) + carry;
        ovf |= scan_write(cnt, g ? gs : bs, g ? gcur : bcur, (r * 1024 + threadIdx.x) * kScanItems, n, off, v[r],
                          g ? cap_g : cap_b);
        carry += tot;
    }
    if (ovf) atomicOr((unsigned long long *)&counters[C_OVERFLOW], g ? 1ull : 2ull);
    if (threadIdx.x == 0) counters[g ? C_GPAIRS : C_BPAIRS] = carry;
}

// ------------------------------------------------------------ scatter

// The pairs of the lanes whose rectangles lie within the 3x3 tiles around
// (cx, cy), the tile of the wave's 8x8 block, for both lists: one cursor
// atomic per (list, neighbouring tile) for the whole wave, all issued by one
// instruction (lane j takes the Gaussian list of tile j, lane 9 + j its
// boundary list) together with the loads of the segments' ends, so the wave
// waits for one round trip; a lane's slot in a tile is the tile's base plus
// its rank among the lanes there (slots past the segment's end, after a
// capacity overflow, are dropped).  Every base and end goes to scalar
// registers before the first key is stored: reading them between the stores
// would make each store wait for the previous one.  Lanes whose rectangle
// reaches further (gin, bin false) are left to the caller.
template <typename EG, typename EB>
__device__ __forceinline__ void near_tiles(bool gin, const TileRect &g, bool bin, const TileRect &b, int cx, int cy,
                                           const ViewInfo &vi, const StatePtrs &st, int lane, EG &&emit_g,
                                           EB &&emit_b) {
    const NearMasks mg(gin, g, cx, cy), mb(bin, b, cx, cy);
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        if (lane == j) cnt = __popcll(mg.at(j));
        if (lane == 9 + j) cnt = __popcll(mb.at(j));
    }
    int base = 0, s0 = 0, c0 = 0;
    if (cnt > 0) {
        const bool isg = lane < 9;
        const int j = isg ? lane : lane - 9;
        const int tl = vi.tile_off + (cy + j / 3 - 1) * vi.tiles_x + cx + j % 3 - 1;
        s0 = (isg ? st.g_start : st.b_start)[tl];
        c0 = (isg ? st.g_count : st.b_count)[tl];
        base = atomicAdd((isg ? st.g_cursor : st.b_cursor) + tl, cnt);
    }
    const int end = s0 + c0;
    int bs[18], es[18];
#pragma unroll
    for (int j = 0; j < 18; ++j) {
        bs[j] = __builtin_amdgcn_readlane(base, j);
        es[j] = __builtin_amdgcn_readlane(end, j);
    }
    auto slot_in = [](unsigned long long m, int first) {  // the lane's rank among the lanes of m, from `first`
        return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, (unsigned)first));
    };
#pragma unroll
    for (int j = 0; j < 9; ++j) {
        const unsigned long long ig = mg.at(j), ib = mb.at(j);
        const int sg = slot_in(ig, bs[j]), sb = slot_in(ib, bs[9 + j]);
        if (__builtin_amdgcn_inverse_ballot_w64(ig) && sg < es[j]) emit_g(sg);
        if (__builtin_amdgcn_inverse_ballot_w64(ib) && sb < es[9 + j]) emit_b(sb);
    }
}

__global__ void __launch_bounds__(256) k_scatter(Consts k, ViewTable vt, StatePtrs st) {
    const int lane = threadIdx.x & 63;
    int v, x, y;
    const int blk = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    const bool act = block8_pixel(vt, blk, lane, v, x, y);
    const ViewInfo vi = vt.v[v];
    const int TSH = __builtin_ctz(k.tile);  // tile side 8, 16 or 32: pixel ranges (>= 0) shift to tiles
    // the tile of the wave's block (x - (lane & 7) is its left edge)
    const int cx = __builtin_amdgcn_readfirstlane((x - (lane & 7)) >> TSH);
    const int cy = __builtin_amdgcn_readfirstlane((y - (lane >> 3)) >> TSH);
    TileRect g, b;
    unsigned long long gkey = 0ull, bkey = 0ull;
    if (act) {
        const int lp = y * vi.W + x, pix = vi.px_off + lp;
        const uint8_t fl = st.pflags[pix];
        if (fl & PF_VALID) {
            // (the three loads in one round trip: the primitive is read for
            // every record, used for boundary points)
            const float4 r3 = st.rec[(int64_t)pix * 4 + 3];
            const unsigned long long depth = st.gkey[pix];
            const int prim = __float_as_int(st.rec[(int64_t)pix * 4 + 2].y);
            const int gx = __float_as_int(r3.x), gy = __float_as_int(r3.y);
            // (in the lattice variant a pixel record is a boundary point only)
            if (k.NL == 0 && lo16(gx) <= hi16(gx) && lo16(gy) <= hi16(gy)) {
                g.x0 = lo16(gx) >> TSH; g.x1 = hi16(gx) >> TSH; g.y0 = lo16(gy) >> TSH; g.y1 = hi16(gy) >> TSH;
            }
            gkey = (depth << 24) | (unsigned long long)lp;
            if (fl & PF_BOUNDARY) {
                const int bx = __float_as_int(r3.z), by = __float_as_int(r3.w);
                if (lo16(bx) <= hi16(bx) && lo16(by) <= hi16(by)) {
                    b.x0 = lo16(bx) >> TSH; b.x1 = hi16(bx) >> TSH; b.y0 = lo16(by) >> TSH; b.y1 = hi16(by) >> TSH;
                }
                bkey = ((unsigned long long)prim << 24) | (unsigned long long)lp;
            }
        }
    }
    // rectangles within the 3x3 tiles around the block's tile (nearly all):
    // one round of cursor atomics for both lists; the rest one cursor atomic
    // per group of lanes at the same tile, each lane taking the slot of its rank
    const bool gnear = g.near(cx, cy), bnear = b.near(cx, cy);
    near_tiles(gnear, g, bnear, b, cx, cy, vi, st, lane, [&](int slot) { st.g_keys[slot] = gkey; },
               [&](int slot) { st.b_keys[slot] = bkey; });
    const unsigned long long below = (1ull << lane) - 1ull;
    if (gnear) g = TileRect();
    if (bnear) b = TileRect();
    for_tiles_grouped(g.x0, g.x1, g.y0, g.y1, vi.tiles_x, vi.tile_off,
                      [&](int t, unsigned long long gm, bool in, int leader) {
        int base = 0;
        if (lane == leader) base = atomicAdd(&st.g_cursor[t], __popcll(gm));
        base = __builtin_amdgcn_readlane(base, leader);
        if (in) {
            const int slot = base + __popcll(gm & below);
            if (slot < st.g_start[t] + st.g_count[t]) st.g_keys[slot] = gkey;
        }
    });
    for_tiles_grouped(b.x0, b.x1, b.y0, b.y1, vi.tiles_x, vi.tile_off,
                      [&](int t, unsigned long long gm, bool in, int leader) {
        int base = 0;
        if (lane == leader) base = atomicAdd(&st.b_cursor[t], __popcll(gm));
        base = __builtin_amdgcn_readlane(base, leader);
        if (in) {
            const int slot = base + __popcll(gm & below);
            if (slot < st.b_start[t] + st.b_count[t]) st.b_keys[slot] = bkey;
        }
    });
}

// Lattice variant: the pairs of the lattice Gaussians, one lane per record;
// a record's key digit is its index within its view, after the view's pixels.
__global__ void __launch_bounds__(256) k_scatter_lattice(Consts k, ViewTable vt, StatePtrs st) {
    const int lane = threadIdx.x & 63;
    const int64_t per_view = (int64_t)k.P * k.NL;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const bool act = i < (int64_t)vt.n * per_view;
    const int v = act ? (int)(i / per_view) : 0;
    const ViewInfo vi = vt.v[v];
    const int TSH = __builtin_ctz(k.tile);  // tile side 8, 16 or 32: pixel ranges (>= 0) shift to tiles
    int gt0 = 1, gt1 = 0, gu0 = 1, gu1 = 0;
    unsigned long long gkey = 0ull;
    if (act) {
        const int64_t rid = vt.total_px + i;
        const float4 r3 = st.rec[rid * 4 + 3];
        const int gx = __float_as_int(r3.x), gy = __float_as_int(r3.y);
        if (lo16(gx) <= hi16(gx) && lo16(gy) <= hi16(gy)) {
            gt0 = lo16(gx) >> TSH; gt1 = hi16(gx) >> TSH; gu0 = lo16(gy) >> TSH; gu1 = hi16(gy) >> TSH;
        }
        const int lr = vi.W * vi.H + (int)(i - v * per_view);
        gkey = (st.gkey[rid] << 24) | (unsigned long long)lr;
    }
    // rectangles within the 3x3 tiles around the middle of the wave's first
    // rectangle (the wave's records are neighbouring nodes of one or two
    // patches), in that rectangle's view: one round of cursor atomics; the
    // rest one cursor atomic per group of lanes at the same tile
    TileRect g;
    g.x0 = gt0; g.x1 = gt1; g.y0 = gu0; g.y1 = gu1;
    const unsigned long long has = __ballot(gt0 <= gt1);
    if (has) {
        const int f = __ffsll((long long)has) - 1;
        const int cx = __builtin_amdgcn_readlane((gt0 + gt1) >> 1, f);
        const int cy = __builtin_amdgcn_readlane((gu0 + gu1) >> 1, f);
        const int vw = __builtin_amdgcn_readlane(v, f);
        const bool near = v == vw && g.near(cx, cy);
        near_tiles(near, g, false, TileRect(), cx, cy, vt.v[vw], st, lane, [&](int slot) { st.g_keys[slot] = gkey; },
                   [&](int) {});
        if (near) g = TileRect();
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    for_tiles_grouped(g.x0, g.x1, g.y0, g.y1, vi.tiles_x, vi.tile_off,
                      [&](int t, unsigned long long gm, bool in, int leader) {
        int base = 0;
        if (lane == leader) base = atomicAdd(&st.g_cursor[t], __popcll(gm));
        base = __builtin_amdgcn_readlane(base, leader);
        if (in) {
            const int slot = base + __popcll(gm & below);
            if (slot < st.g_start[t] + st.g_count[t]) st.g_keys[slot] = gkey;
        }
    });
}

// ------------------------------------------------------------ segment sort

// Ascending bitonic network whose first step of every merge compares mirrored
// positions; positions >= n behave as +inf and never move, so a segment is
// padded virtually to the next power of two.
template <typename CmpX>
__device__ __forceinline__ void bitonic_steps(int n2, CmpX cmpx) {
    for (int kk = 2; kk <= n2; kk <<= 1) {
        const int half = kk >> 1;
        for (int q = threadIdx.x; q < (n2 >> 1); q += blockDim.x) {
            const int blk = q / half, pos = q % half;
            cmpx(blk * kk + pos, blk * kk + kk - 1 - pos);
        }
        __syncthreads();
        for (int j = kk >> 2; j >= 1; j >>= 1) {
            for (int q = threadIdx.x; q < (n2 >> 1); q += blockDim.x) {
                const int blk = q / j, pos = q % j;
                const int a = blk * 2 * j + pos;
                cmpx(a, a + j);
            }
            __syncthreads();
        }
    }
}

// The list positions of tile t (of view v) under its slot: gpos[rec] is
// the position of record rec in the tile's list.
__device__ __forceinline__ int32_t *list_positions(const ViewTable &vt, const StatePtrs &st, int v, int t) {
    const int tl = t - vt.v[v].tile_off, tx = tl % vt.v[v].tiles_x, ty = tl / vt.v[v].tiles_x;
    return st.gpos + (int64_t)tile_slot(tx, ty) * st.n_rec;
}

// The key of lane l ^ m (m a power of two below 64): DPP within quads
// (plain VALU moves), an LDS swizzle within 32-lane halves, a permute across
// them.
__device__ __forceinline__ int xor_lane(int v, int m) {
    if (m == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);  // quad_perm [1, 0, 3, 2]
    if (m == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);  // quad_perm [2, 3, 0, 1]
    if (m == 4) return __builtin_amdgcn_ds_swizzle(v, 0x101F);               // bit mode: and 31, xor 4
    if (m == 8) return __builtin_amdgcn_ds_swizzle(v, 0x201F);
    if (m == 16) return __builtin_amdgcn_ds_swizzle(v, 0x401F);
    return __shfl_xor(v, m, 64);
}
__device__ __forceinline__ unsigned long long xor_lane(unsigned long long v, int m) {
    const int lo = xor_lane((int)(unsigned)v, m), hi = xor_lane((int)(unsigned)(v >> 32), m);
    return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
}

// Ascending bitonic sort of the 64 R keys x[r] of lane l (key l R + r)
// across the wave: partners fewer than R apart are in the same lane, the
// others (fewer steps) are exchanged between lanes.  Padding keys (~0) sort
// last.
template <int R>
__device__ __forceinline__ void wave_sort_regs(unsigned long long (&x)[R], int lane) {
#pragma unroll
    for (int k = 2; k <= 64 * R; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j >= 1; j >>= 1) {
            if (j < R) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int r2 = r ^ j;
                    if (r2 < r) continue;
                    // ascending where bit k of the key index l R + r is clear
                    const bool up = (((lane * R) | r) & k) == 0;
                    const unsigned long long a = x[r], b = x[r2];
                    const bool sw = (b < a) == up;  // (equal keys: either)
                    x[r] = sw ? b : a;
                    x[r2] = sw ? a : b;
                }
            } else {
                const int m = j / R;  // partner lane l ^ m
                // the lower lane of a pair keeps the smaller key in ascending
                // runs: it takes the partner's key when that is smaller, the
                // upper lane when it is larger (equal keys: either)
                const bool keep_min = ((lane & m) == 0) == (((lane * R) & k) == 0);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const unsigned long long y = xor_lane(x[r], m);
                    x[r] = (y < x[r]) == keep_min ? y : x[r];
                }
            }
        }
    }
}

// Lists up to this length are sorted by one wave in registers; longer ones
// are queued for a workgroup each.
constexpr int kWaveSort = 512;

// LDS slot of key i of a wave's staging buffer: 8 bytes of padding after
// every 8 keys, so that lanes reading 8 consecutive keys each hit distinct
// banks
__device__ __forceinline__ int stage_slot(int i) { return i + (i >> 3); }
constexpr int kStageKeys = kWaveSort + kWaveSort / 8;

// Sorts one list of cnt <= 64 R keys.  Multi-key lanes load and store
// through the wave's LDS buffer sb, so that global memory is read and written
// in 64-lane runs while each lane sorts consecutive keys.
template <int R, typename Emit>
__device__ __forceinline__ void wave_sort_list(const unsigned long long *src, int cnt, int lane, unsigned long long *sb,
                                               Emit &&emit) {
    unsigned long long x[R];
    if constexpr (R == 1) {
        x[0] = lane < cnt ? src[lane] : ~0ull;
        wave_sort_regs<1>(x, lane);
        if (lane < cnt) emit(lane, x[0]);
        return;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * 64 + lane;
        sb[stage_slot(i)] = i < cnt ? src[i] : ~0ull;
    }
    // (one wave's LDS accesses complete in order: the fence keeps the
    // compiler from moving them across each other)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = sb[stage_slot(lane * R + r)];
    wave_sort_regs<R>(x, lane);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) sb[stage_slot(lane * R + r)] = x[r];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * 64 + lane;
        if (i < cnt) emit(i, sb[stage_slot(i)]);
    }
}

// Sorts one list of 256 < cnt <= 256 + 64 RB keys without sorting padding up
// to 512: the first 256 keys (4 per lane) and the rest (RB per lane) are
// sorted in registers as two runs, then merged along the merge path, each
// lane writing per = ceil(cnt / 64) consecutive outputs: a binary search
// finds how many of them come from the first run, then one comparison per
// output walks both runs (keys of the first run go before equal keys of the
// second).
template <int RB, typename Emit>
__device__ __forceinline__ void wave_sort_split(const unsigned long long *src, int cnt, int lane,
                                                unsigned long long *sb, Emit &&emit) {
    constexpr int RA = 4, NA = 64 * RA;
    unsigned long long x[RA], y[RB];
#pragma unroll
    for (int r = 0; r < RA + RB; ++r) {
        const int i = r * 64 + lane;
        sb[stage_slot(i)] = i < cnt ? src[i] : ~0ull;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < RA; ++r) x[r] = sb[stage_slot(lane * RA + r)];
#pragma unroll
    for (int r = 0; r < RB; ++r) y[r] = sb[stage_slot(NA + lane * RB + r)];
    wave_sort_regs<RA>(x, lane);
    wave_sort_regs<RB>(y, lane);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < RA; ++r) sb[stage_slot(lane * RA + r)] = x[r];
#pragma unroll
    for (int r = 0; r < RB; ++r) sb[stage_slot(NA + lane * RB + r)] = y[r];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int lb = cnt - NA, per = (cnt + 63) >> 6, d = lane * per;
    if (d >= cnt) return;
    int lo = max(0, d - lb), hi = min(d, NA);
    while (lo < hi) {
        const int c = (lo + hi) >> 1;
        if (sb[stage_slot(c)] <= sb[stage_slot(NA + d - 1 - c)]) lo = c + 1;
        else hi = c;
    }
    int i = lo, j = d - lo;
    // (a read one past the first run is the second run's first key, one past
    // the second a padding slot; neither is taken)
    unsigned long long ka = sb[stage_slot(i)], kb = sb[stage_slot(NA + j)];
    const int m = min(per, cnt - d);
#pragma unroll
    for (int k = 0; k < RA + RB; ++k)
        if (k < m) {
            const bool take_a = i < NA && (j >= lb || ka <= kb);
            emit(d + k, take_a ? ka : kb);
            i += take_a;
            j += !take_a;
            const unsigned long long nx = sb[stage_slot(take_a ? i : NA + j)];
            ka = take_a ? nx : ka;
            kb = take_a ? kb : nx;
        }
}

// One wave per list: list L < n_tiles is the Gaussian list of tile L, the
// others the boundary lists.  Empty lists cost a wave a few instructions.
// The first thread also copies the pass's overflow bits (complete since the
// scan), when there are any, into the context's word of pinned host memory: a
// later call on the context (and bgt_query) reads it without waiting for the
// device.  A plain system-scope store, not an atomic, so nothing depends on the
// host bridge's atomics.
__global__ void __launch_bounds__(256) k_sort_lists(ViewTable vt, StatePtrs st, int lat_per_view,
                                                    unsigned long long *flag) {
    __shared__ unsigned long long stage[4][kStageKeys];
    const int lane = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x == 0 && flag) {
        const unsigned long long f = (unsigned long long)st.counters[C_OVERFLOW];
        if (f) __hip_atomic_store(flag, f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    const int L = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (L >= 2 * vt.total_tiles) return;
    const int which = L < vt.total_tiles ? 0 : 1, t = which == 0 ? L : L - vt.total_tiles;
    const int cnt = which == 0 ? st.g_count[t] : st.b_count[t];
    if (cnt == 0 || cnt > kWaveSort) return;  // (longer lists: k_sort_long)
    const int start = which == 0 ? st.g_start[t] : st.b_start[t];
    const unsigned long long *src = (which == 0 ? st.g_keys : st.b_keys) + start;
    const int v = view_of_tile(vt, t);
    uint32_t *dst = (which == 0 ? st.g_list : st.b_list) + start;
    // a Gaussian list also records each entry's position under its record's
    // tile slot, for the parameter pass
    int32_t *gpos = which == 0 ? list_positions(vt, st, v, t) : nullptr;
    auto emit = [&](int i, unsigned long long key) {
        const int rec = record_of(vt, v, (int)(key & 0xFFFFFFull), lat_per_view);
        dst[i] = (uint32_t)rec;
        if (gpos) gpos[rec] = start + i;
    };
    unsigned long long *sb = stage[threadIdx.x >> 6];
    if (cnt <= 64) wave_sort_list<1>(src, cnt, lane, sb, emit);
    else if (cnt <= 128) wave_sort_list<2>(src, cnt, lane, sb, emit);
    else if (cnt <= 256) wave_sort_list<4>(src, cnt, lane, sb, emit);
    else if (cnt <= 320) wave_sort_split<1>(src, cnt, lane, sb, emit);
    else if (cnt <= 384) wave_sort_split<2>(src, cnt, lane, sb, emit);
    else wave_sort_list<8>(src, cnt, lane, sb, emit);
}

// Lists longer than a wave sorts, one workgroup per list: workgroup b takes
// the long lists among `chunk` tiles, whose counts its threads read at
// once (no queue, no global atomic).  Tile i of the launch is tile
// i (2^31 - 1) mod n, a permutation (2^31 - 1 is a prime above n) that
// spreads the long lists, which cluster in neighbouring tiles and at the
// same place in similar views, over the workgroups.  Up to kSortLds keys:
// runs of kWaveSort keys sorted in registers, one wave per run (padded with
// ~0, above every key), then merged pairwise, level by level.  A thread
// writes `per` consecutive outputs of a level (a power of two, at most
// kSortLds / 256): a binary search along the merge path finds how many of
// them come from the pair's first run, then one comparison per output walks
// both runs (keys of the first run go before equal keys of the second).  In
// place: every thread merges its outputs into registers first and all write
// after a barrier, so the block needs one buffer (18 KB); the last level's
// outputs go to the list at once.
// Longer lists, up to kRankRuns such buffers: each kSortLds keys sorted so in
// place, then a key's position is its index in its own run plus the number of
// smaller keys in each of the others (keys are unique), found by binary search
// in LDS, eight keys of a thread at a time, about 6 us per pair of runs.  Beyond
// that (a correctness path) a bitonic network in global memory, whose steps
// each wait for memory but whose work grows less than quadratically: at 30
// runs it is the faster one (3.9 against 5.3 ms for the scene below).
// What bounds it is the latency of one list: 90 -> 27 us for 8000 patches in a
// 1000x1000 view with tiles of 16, 72 -> 22 us for three views near 701x523, both
// by one list per workgroup instead of several; 16 -> 3.9 ms with 334 lists
// beyond the buffer (2880 patches' lattice Gaussians, 14 views of 144x144).
constexpr int kLongChunk = 16;  // the most tiles per workgroup
constexpr int kRankRuns = 16;
constexpr int kLongGroups = 2560;  // see launch_binning
static_assert(kSortLds == 4 * kWaveSort, "the four waves of a workgroup sort one run each");

// Sorts src[0, cnt), cnt <= kSortLds, by a workgroup of 256 threads;
// out(i, key) takes the i-th smallest.  Every key is read before the first
// call of out.
template <typename Out>
__device__ __forceinline__ void block_sort(const unsigned long long *src, int cnt, unsigned long long *keys, Out &&out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // runs of 512 keys, one wave each: loaded into the buffer in 64-lane
    // runs (a thread's loads all in flight), read by each lane as 8
    // consecutive keys, sorted in registers
    {
        unsigned long long x[kSortLds / 256];
#pragma unroll
        for (int r = 0; r < kSortLds / 256; ++r) {
            const int i = r * 256 + (int)threadIdx.x;
            x[r] = i < cnt ? src[i] : 0ull;
        }
#pragma unroll
        for (int r = 0; r < kSortLds / 256; ++r) {
            const int i = r * 256 + (int)threadIdx.x;
            if (i < cnt) keys[stage_slot(i)] = x[r];
        }
    }
    __syncthreads();
    if (wave * kWaveSort < cnt) {
        unsigned long long x[8];
        const int b0 = wave * kWaveSort + lane * 8;
#pragma unroll
        for (int r = 0; r < 8; ++r) x[r] = b0 + r < cnt ? keys[stage_slot(b0 + r)] : ~0ull;
        wave_sort_regs<8>(x, lane);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (b0 + r < cnt) keys[stage_slot(b0 + r)] = x[r];
    }
    __syncthreads();
    if (cnt <= kWaveSort)  // (the end of a longer list: one run, nothing to merge)
        for (int i = threadIdx.x; i < cnt; i += blockDim.x) out(i, keys[stage_slot(i)]);
    // outputs per thread: a power of two, so that no thread's outputs
    // straddle two pairs of runs
    int per = 1;
    while (per * 256 < cnt) per <<= 1;
    for (int L = kWaveSort; L < cnt; L <<= 1) {
        unsigned long long x[kSortLds / 256];
        const int d0 = threadIdx.x * per;
        int m = 0;
        if (d0 < cnt) {
            const int p0 = d0 & ~(2 * L - 1);
            const int mid = min(p0 + L, cnt), end = min(p0 + 2 * L, cnt);
            const int la = mid - p0, lb = end - mid, d = d0 - p0;
            // how many of the pair's first d outputs come from the first
            // run (the first run's keys go before equal keys of the second)
            int lo = max(0, d - lb), hi = min(d, la);
            while (lo < hi) {
                const int c = (lo + hi) >> 1;
                if (keys[stage_slot(p0 + c)] <= keys[stage_slot(mid + d - 1 - c)]) lo = c + 1;
                else hi = c;
            }
            int i = lo, j = d - lo;
            // (reads one past a run's end stay in the buffer, which has a
            // slot past the last key; their values are never taken)
            unsigned long long ka = keys[stage_slot(p0 + i)], kb = keys[stage_slot(mid + j)];
            m = min(per, end - d0);
#pragma unroll
            for (int k = 0; k < kSortLds / 256; ++k)
                if (k < m) {
                    const bool take_a = i < la && (j >= lb || ka <= kb);
                    x[k] = take_a ? ka : kb;
                    i += take_a;
                    j += !take_a;
                    const unsigned long long nx = keys[stage_slot(take_a ? p0 + i : mid + j)];
                    ka = take_a ? nx : ka;
                    kb = take_a ? kb : nx;
                }
        }
        if (2 * L >= cnt) {  // the last level
#pragma unroll
            for (int k = 0; k < kSortLds / 256; ++k)
                if (k < m) out(d0 + k, x[k]);
        } else {  // in place: all read, then all write
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kSortLds / 256; ++k)
                if (k < m) keys[stage_slot(d0 + k)] = x[k];
            __syncthreads();
        }
    }
    __syncthreads();  // the next use of the buffer
}

// Positions of the keys of the runs src[kSortLds r, kSortLds (r + 1)), each
// sorted, in the order of all of them: out(i, key).
template <typename Out>
__device__ __forceinline__ void block_rank_runs(const unsigned long long *src, int cnt, unsigned long long *keys,
                                                Out &&out) {
    constexpr int R = kSortLds / 256;
    auto load = [&](int b0, unsigned long long *y) {  // (a thread's loads all in flight)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = b0 + r * 256 + (int)threadIdx.x;
            y[r] = i < cnt ? src[i] : ~0ull;
        }
    };
    for (int a0 = 0; a0 < cnt; a0 += kSortLds) {
        const int na = min(kSortLds, cnt - a0);
        unsigned long long x[R], y[R];
        int rank[R];
        load(a0, x);
#pragma unroll
        for (int r = 0; r < R; ++r) rank[r] = r * 256 + (int)threadIdx.x;
        int b0 = a0 == 0 ? kSortLds : 0;
        load(b0, y);
        while (b0 < cnt) {
            const int nb = min(kSortLds, cnt - b0);
#pragma unroll
            for (int r = 0; r < R; ++r) keys[stage_slot(r * 256 + (int)threadIdx.x)] = y[r];
            __syncthreads();
            b0 += b0 + kSortLds == a0 ? 2 * kSortLds : kSortLds;
            load(b0, y);  // (the next run is on its way during the search)
            int pos[R];
#pragma unroll
            for (int r = 0; r < R; ++r) pos[r] = 0;
            for (int step = kSortLds; step > 0; step >>= 1)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int q = min(pos[r] + step, kSortLds);
                    pos[r] = pos[r] + step <= nb && keys[stage_slot(q - 1)] < x[r] ? q : pos[r];
                }
#pragma unroll
            for (int r = 0; r < R; ++r) rank[r] += pos[r];
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r * 256 + (int)threadIdx.x < na) out(rank[r], x[r]);
    }
}

__global__ void __launch_bounds__(256, 5) k_sort_long(ViewTable vt, StatePtrs st, int lat_per_view, int chunk) {
    __shared__ unsigned long long keys[kSortLds + kSortLds / 8 + 1];
    __shared__ int long_tiles[kLongChunk], n_long;
    const int which = blockIdx.y;
    if (threadIdx.x == 0) n_long = 0;
    __syncthreads();
    if ((int)threadIdx.x < chunk) {
        const int i = blockIdx.x * chunk + threadIdx.x;
        if (i < vt.total_tiles) {
            const int t = (int)((int64_t)i * 2147483647ll % vt.total_tiles);
            if ((which == 0 ? st.g_count[t] : st.b_count[t]) > kWaveSort) long_tiles[atomicAdd(&n_long, 1)] = t;
        }
    }
    __syncthreads();
    for (int li = 0; li < n_long; ++li) {
        const int t = long_tiles[li];
        const int cnt = which == 0 ? st.g_count[t] : st.b_count[t];
        const int start = which == 0 ? st.g_start[t] : st.b_start[t];
        unsigned long long *src = (which == 0 ? st.g_keys : st.b_keys) + start;
        const int v = view_of_tile(vt, t);
        uint32_t *dst = (which == 0 ? st.g_list : st.b_list) + start;
        int32_t *gpos = which == 0 ? list_positions(vt, st, v, t) : nullptr;
        auto emit = [&](int i, unsigned long long key) {
            const int rec = record_of(vt, v, (int)(key & 0xFFFFFFull), lat_per_view);
            dst[i] = (uint32_t)rec;
            if (gpos) gpos[rec] = start + i;
        };
        if (cnt <= kSortLds) {
            block_sort(src, cnt, keys, emit);
            continue;
        }
        if (threadIdx.x == 0) atomicAdd((unsigned long long *)&st.counters[C_BIGSORT], 1ull);
        if (cnt <= kRankRuns * kSortLds) {
            for (int r = 0; r < cnt; r += kSortLds)
                block_sort(src + r, min(kSortLds, cnt - r), keys, [&](int i, unsigned long long key) { src[r + i] = key; });
            block_rank_runs(src, cnt, keys, emit);
        } else {
            int n2 = 1;
            while (n2 < cnt) n2 <<= 1;
            bitonic_steps(n2, [&](int a, int b) {
                if (b >= cnt) return;
                const unsigned long long x = src[a], y = src[b];
                if (y < x) { src[a] = y; src[b] = x; }
            });
            for (int i = threadIdx.x; i < cnt; i += blockDim.x) emit(i, src[i]);
        }
        __syncthreads();
    }
}

hipError_t launch_binning(const Consts &k, const ViewTable &vt, const StatePtrs &st, unsigned long long *flag,
                          hipStream_t s) {
    const int n = vt.total_tiles;
    if (n <= kScanOne) {
        hipLaunchKernelGGL(k_scan_one, dim3(3), dim3(1024), 0, s, st.g_count, st.g_start, st.g_cursor, st.b_count,
                           st.b_start, st.b_cursor, n, k.cap_g, k.cap_b, st.counters, st.order);
    } else {
        int32_t *classes = (int32_t *)(st.counters + kOrderWord);
        const int nb = (n + kScanBlock - 1) / kScanBlock;
        int64_t *sums = (int64_t *)st.scan_tmp;
        hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kScanThreads), 0, s, (const int32_t *)st.g_count,
                           (const int32_t *)st.b_count, n, sums, nb, classes);
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, sums, nb, st.counters, classes);
        hipLaunchKernelGGL(k_scan_down, dim3(nb), dim3(kScanThreads), 0, s, st.g_count, st.g_start, st.g_cursor,
                           st.b_count, st.b_start, st.b_cursor, (const int64_t *)sums, n, nb, k.cap_g, k.cap_b,
                           st.counters, classes, st.order);
    }
    hipLaunchKernelGGL(k_scatter, dim3((unsigned)((vt.total_b8 + 3) / 4)), dim3(256), 0, s, k, vt, st);
    const int lat_per_view = k.P * k.NL;
    if (lat_per_view > 0) {
        const int64_t nl = (int64_t)vt.n * lat_per_view;
        hipLaunchKernelGGL(k_scatter_lattice, dim3((unsigned)((nl + 255) / 256)), dim3(256), 0, s, k, vt, st);
    }
    hipLaunchKernelGGL(k_sort_lists, dim3((unsigned)((2 * (int64_t)n + 3) / 4)), dim3(256), 0, s, vt, st,
                       lat_per_view, flag);
    // Tiles per workgroup of the long lists: one, so that no workgroup sorts
    // several lists one after the other, up to kLongGroups tiles; beyond, more
    // tiles, since nearly all of the workgroups would only find that they have no
    // long list.  The chip holds 1280 of these workgroups at once (five per CU by
    // their registers), so the line is not where they all fit but a measured one, in
    // us at 1 / 2 / 4 / 16 tiles per workgroup: 2500 tiles with long lists (8000
    // cubic patches, 800x800, 16 px) 18 / 24 / - / 45, 3969 (the same at 1000x1000)
    // 22 / 28 / 40 / 94, against 10000 with hardly any (2000 patches, 8 px) 12 / 7 / 5 / 5.
    int chunk = 1;
    while (chunk < kLongChunk && n / chunk > kLongGroups) chunk <<= 1;
    hipLaunchKernelGGL(k_sort_long, dim3((unsigned)((n + chunk - 1) / chunk), 2), dim3(256), 0, s, vt, st,
                       lat_per_view, chunk);
    return hipGetLastError();
}

}  // namespace bgt
