// HIP kernels of the FRNN graph builder for CDNA4 (gfx950, wave64).
//
// Pipeline of one call (paper, Section 3.4: bin the points by three projected
// coordinates into grid cells, then visit only the cells around each query):
//   k_bounds      min/max of the binned coordinates and a non-finite check over
//                 all coordinates; clears what the call counts in
//   k_bin         grid plan (cell edge, cells per axis), cell of every point, each share
//                 of points sorted by tile (a run of cells) in LDS
//   k_tiles       each tile's points gathered from the shares, counted and ordered by
//                 cell in LDS: first sorted row of each cell, the search's shares of equal
//                 work (cells' fixed costs plus queries), rows copied into cell order;
//                 tiles of many points by several workgroups
//   or, for calls with an event of more than kBinMaxRows rows, in place of the two:
//   k_keys        grid plan, cell key of every point, histogram with in-cell arrival
//                 rank, per-tile histogram totals
//   k_scan_cells  exclusive scan of the histogram -> first sorted row of each cell;
//                 the search's shares of equal work
//   k_scatter     counting-sort scatter: rows copied into cell order
//   k_search      each wave takes a share of equal work in cell order: a
//                 cell's queries against the (2R+1)^(axes-1) contiguous runs of
//                 neighbouring cells along axis 0; each lane holds one candidate (its
//                 leading coordinates, two to four), those of the query are
//                 wave-uniform; an exact early exit after as many terms of the
//                 distance sum; ballots queue the survivors, whose sums are finished 64 at a
//                 time; the lists of pending queries are stored as found, in batches
//   k_kept_sums   kept totals per placement tile and per group of tiles
//   k_place       output offsets from the totals and a block scan; each short list
//                 sorted by its query's thread and the block's output formed in LDS,
//                 then written to its (i asc, j asc) positions with coalesced
//                 stores; then the queued lists longer than the search keeps, or
//                 longer than K, collected again, one per wave at a time (the K smallest
//                 by (D, j) found bit by bit with ballots), those of more than kWaveKeys
//                 hits one per workgroup (MSB-first radix select)
//
// Distances follow one fixed order with every product and sum rounded on its
// own: this file is compiled with -ffp-contract=off and the pragma below.

#include <float.h>

#include <algorithm>

#include "frnn_internal.h"

#pragma clang fp contract(off)

namespace frnn {
namespace {

// base plus the set bits below the lane's own.
__device__ __forceinline__ unsigned int prefix_count(unsigned long long mask, unsigned int base = 0u) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<unsigned int>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<unsigned int>(mask), base));
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
// Neighbours kept, from a query's kept word.
__device__ __forceinline__ unsigned int kept_count(unsigned int w) {
    return w & ((w & kKeptExt) != 0u ? kKeptExtCount : ~kKeptLong);
}
// Wave index inside the workgroup, marked wave-uniform for the compiler (so that
// values derived from it live in scalar registers and feed scalar loads).
__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
}

__device__ __forceinline__ unsigned int uniform(unsigned int v) { return __builtin_amdgcn_readfirstlane(v); }

// Orders the LDS accesses of one wave (lanes of a wave exchange data through LDS
// without a workgroup barrier).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Partial sum of the definition over coordinates [K0, K1): ascending order, every
// product and sum rounded on its own.  Rows are zero-padded; adding +0 leaves a
// sum unchanged, so padded rows give the same D as unpadded ones.  Partial sums of
// non-negative terms never decrease, so s >= r2 after a prefix rejects exactly.
template <int K0, int K1, int DP, int NB>
__device__ __forceinline__ float add_terms(float s, const float (&a)[DP], const float (&b)[NB]) {
#pragma unroll
    for (int k = K0; k < K1; ++k) {
        const float t = a[k] - b[k];
        const float t2 = t * t;
        s = s + t2;
    }
    return s;
}

template <int DP>
__device__ __forceinline__ float sq_dist(const float (&a)[DP], const float (&b)[DP]) {
    return add_terms<0, DP, DP, DP>(0.0f, a, b);
}

// Terms before the first exact rejection test of the search: two for rows of up to 12
// floats (a three-term test rejects few more pairs than two terms do, and the first
// stage runs for every query and candidate; on the 300k-point 12-D event two, three and
// four terms took 87.5, 88.7 and 89.6 us), three for rows of 16 and 24 floats, four for
// wider ones (two terms took whole 120k-point builds with 32-, 48- and 64-float rows from
// 0.173, 0.292 and 0.558 ms to 0.204, 0.423 and 1.126 ms).
constexpr int search_lead(int dpad) { return dpad <= 12 ? 2 : (dpad < 32 ? 3 : 4); }

// The sorted points, zero-padded to DP coordinates (a multiple of 4).  Rows of 12 floats
// and more lie in two parts: the first four coordinates of all rows, of which the search's
// first stage reads two to four for every candidate, side by side (16 bytes a row instead
// of a line or a good part of one each), then the rest of each row.  Whole builds with
// whole and with split rows: 300k points of 12 coordinates 129.8 and 127.1 us, 60k of 16
// 55.5 and 54.2, of 32, 48 and 64 95, 88.7 and 121.7 against 88, 85.7 and 103.8; with rows
// of 8 a dense 60k-point event 122.8 and 124.8, a batch of 5.6M points 1416 and 1424.
constexpr int kSplitFrom = 12;

template <int DP>
struct SortedRows {
    static constexpr bool kSplit = DP >= kSplitFrom;
    static constexpr int kLead = search_lead(DP);
    static constexpr int kHead = kSplit ? 4 : kLead;  // coordinates in the leading part
    static constexpr int kTail = DP - kLead;          // coordinates of the second stage
    static constexpr int kLeadStride = kSplit ? kHead : DP;
    static constexpr int kRestStride = kSplit ? DP - kHead : DP;
    const float *__restrict__ lead;
    const float *__restrict__ rest;
    static __device__ __forceinline__ size_t rest_at(long long rows) {
        return kSplit ? static_cast<size_t>(rows) * kHead : static_cast<size_t>(kHead);
    }
    __device__ __forceinline__ SortedRows(const float *__restrict__ sorted, long long rows)
        : lead(sorted), rest(sorted + rest_at(rows)) {}
    __device__ __forceinline__ const float *lead_of(unsigned int s) const {
        return lead + static_cast<size_t>(s) * kLeadStride;
    }
    __device__ __forceinline__ float at(unsigned int s, int k) const {
        return k < kHead ? lead_of(s)[k] : rest[static_cast<size_t>(s) * kRestStride + (k - kHead)];
    }
    // Coordinates from FROM on.
    template <int FROM>
    __device__ __forceinline__ void load(unsigned int s, float (&c)[DP]) const {
        const float *a = lead_of(s), *b = rest + static_cast<size_t>(s) * kRestStride;
#pragma unroll
        for (int k = FROM; k < kHead; ++k) c[k] = a[k];
#pragma unroll
        for (int k = FROM > kHead ? FROM : kHead; k < DP; ++k) c[k] = b[k - kHead];
    }
    static __device__ __forceinline__ void store(float *__restrict__ sorted, long long rows, unsigned int s,
                                                 const float (&c)[DP]) {
        float *a = sorted + static_cast<size_t>(s) * kLeadStride;
        float *b = sorted + rest_at(rows) + static_cast<size_t>(s) * kRestStride;
#pragma unroll
        for (int k = 0; k < kHead; ++k) a[k] = c[k];
#pragma unroll
        for (int k = kHead; k < DP; ++k) b[k - kHead] = c[k];
    }
};

// Cross-lane steps with DPP (GFX9 encodings): row_shr:n moves lane i - n of the
// same 16-lane row into lane i (0 when that lane is in another row); row_bcast:15
// gives the rows selected by the row mask lane 15 of the row before; row_bcast:31
// gives them lane 31.  Rows the mask leaves out keep `old` (here 0).
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ unsigned int dpp_move(unsigned int v) {
    return static_cast<unsigned int>(
        __builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROW_MASK, 0xf, true));
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ unsigned long long dpp_move(unsigned long long v) {
    const unsigned int lo = dpp_move<CTRL, ROW_MASK>(static_cast<unsigned int>(v));
    const unsigned int hi = dpp_move<CTRL, ROW_MASK>(static_cast<unsigned int>(v >> 32));
    return static_cast<unsigned long long>(hi) << 32 | lo;
}
// The same moves for a min/max fold: lanes without a source keep their own value.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_keep(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROW_MASK, 0xf,
                                                      false));
}
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;
constexpr int kWaveShr1 = 0x138;  // lane i - 1 of the whole wave (0 in lane 0)

// Inclusive prefix sum across the 64 lanes (a scan within each row of 16 lanes,
// then the row totals carried into the rows after them), for 32- or 64-bit
// unsigned values.
template <typename T>
__device__ __forceinline__ T wave_scan_add(T x) {
    x += dpp_move<kRowShr1>(x);
    x += dpp_move<kRowShr2>(x);
    x += dpp_move<kRowShr4>(x);
    x += dpp_move<kRowShr8>(x);
    x += dpp_move<kRowBcast15, 0xa>(x);
    x += dpp_move<kRowBcast31, 0xc>(x);
    return x;
}

// Value of lane 63 in every lane.
__device__ __forceinline__ unsigned int lane63(unsigned int x) { return __builtin_amdgcn_readlane(x, 63); }
__device__ __forceinline__ unsigned long long lane63(unsigned long long x) {
    return static_cast<unsigned long long>(__builtin_amdgcn_readlane(static_cast<unsigned int>(x >> 32), 63)) << 32 |
           __builtin_amdgcn_readlane(static_cast<unsigned int>(x), 63);
}
__device__ __forceinline__ float lane63(float x) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// Sum over the 64 lanes, in every lane (32- or 64-bit unsigned).
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    return lane63(wave_scan_add(v));
}

// Inclusive prefix sum across the 64 lanes of a wave.
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v) {
    return wave_scan_add(v);
}

// Minimum and maximum over the 64 lanes, in every lane.
__device__ __forceinline__ float wave_min(float x) {
    x = fminf(x, dpp_keep<kRowShr1>(x));
    x = fminf(x, dpp_keep<kRowShr2>(x));
    x = fminf(x, dpp_keep<kRowShr4>(x));
    x = fminf(x, dpp_keep<kRowShr8>(x));
    x = fminf(x, dpp_keep<kRowBcast15, 0xa>(x));
    x = fminf(x, dpp_keep<kRowBcast31, 0xc>(x));
    return lane63(x);
}
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp_keep<kRowShr1>(x));
    x = fmaxf(x, dpp_keep<kRowShr2>(x));
    x = fmaxf(x, dpp_keep<kRowShr4>(x));
    x = fmaxf(x, dpp_keep<kRowShr8>(x));
    x = fmaxf(x, dpp_keep<kRowBcast15, 0xa>(x));
    x = fmaxf(x, dpp_keep<kRowBcast31, 0xc>(x));
    return lane63(x);
}
__device__ __forceinline__ int wave_any(int x) { return __builtin_amdgcn_ballot_w64(x != 0) != 0ull ? 1 : 0; }

// Sum over the block; every thread gets the total.
__device__ unsigned long long block_sum(unsigned long long v, unsigned long long *scratch) {
    v = wave_sum(v);
    if (lane_id() == 0) scratch[wave_id()] = v;
    __syncthreads();
    unsigned long long t = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) t += scratch[w];
    __syncthreads();
    return t;
}

// Exclusive prefix over the block in thread order.
__device__ unsigned long long block_exclusive_scan(unsigned long long v, unsigned long long *scratch) {
    unsigned long long inc = wave_inclusive_scan(v);
    if (lane_id() == 63) scratch[wave_id()] = inc;
    __syncthreads();
    unsigned long long before = 0;
    for (int w = 0; w < wave_id(); ++w) before += scratch[w];
    __syncthreads();
    return before + inc - v;
}

// Block sums of a and b and the exclusive prefix of c in thread order, with one
// barrier: red (3 kWaves entries) belongs to this call alone, so it needs no
// barrier after it.
__device__ void block_sums_and_scan(unsigned long long a, unsigned long long b, unsigned long long c,
                                    unsigned long long *red, unsigned long long &sum_a, unsigned long long &sum_b,
                                    unsigned long long &before_c) {
    a = wave_sum(a);
    b = wave_sum(b);
    const unsigned long long inc = wave_inclusive_scan(c);
    if (lane_id() == 63) {
        red[wave_id()] = a;
        red[kWaves + wave_id()] = b;
        red[2 * kWaves + wave_id()] = inc;
    }
    __syncthreads();
    unsigned long long sa = 0, sb = 0, pre = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        sa += red[w];
        sb += red[kWaves + w];
        pre += w < wave_id() ? red[2 * kWaves + w] : 0ull;
    }
    sum_a = sa;
    sum_b = sb;
    before_c = pre + inc - c;
}

// ------------------------------------------------------------------ bounds

// Binned coordinates of an event, axis 0 first; -1 for an axis that is not binned.
struct Dims {
    int c[kMaxAxes];
};

// Minimum and maximum of N columns that a thread sees, and whether a value was not a
// number (infinite values show in the minimum or maximum).
template <int N>
struct BoundsAcc {
    float mn[N], mx[N];
    bool nan = false;
    __device__ __forceinline__ BoundsAcc() {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            mn[k] = INFINITY;
            mx[k] = -INFINITY;
        }
    }
    __device__ __forceinline__ void add(int k, float v) {
        nan |= v != v;
        mn[k] = fminf(mn[k], v);
        mx[k] = fmaxf(mx[k], v);
    }
    __device__ __forceinline__ bool bad() const {
        bool b = nan;
#pragma unroll
        for (int k = 0; k < N; ++k) b |= mn[k] == -INFINITY || mx[k] == INFINITY;
        return b;
    }
};

// Grid (bounds blocks, n_events): block (b, e) folds a share of event e's rows.
// The first blocks also clear the counters of the call and what its binning counts in: the
// histogram and the tile totals, or the crowded tiles' counts and their sums.
__global__ __launch_bounds__(kBlock) void k_bounds(int d, Dims dd,
                                                   int vec4, EventDesc *__restrict__ ev, EventDesc ev0,
                                                   int ev_from_arg, BoundsPartial *__restrict__ part,
                                                   unsigned int *__restrict__ counts, long long n_counts,
                                                   unsigned long long *__restrict__ sums, int n_sums,
                                                   Counters *__restrict__ ctr) {
    const long long nblk = static_cast<long long>(gridDim.x) * gridDim.y;
    const long long bid = static_cast<long long>(blockIdx.y) * gridDim.x + blockIdx.x;
    const long long gtid = bid * kBlock + threadIdx.x;
    const long long gstride = nblk * kBlock;
    for (long long c = gtid; c < n_counts; c += gstride) counts[c] = 0u;
    for (long long c = gtid; c < n_sums; c += gstride) sums[c] = 0ull;
    if (gtid == 0) {
        Counters z = {};
        *ctr = z;
        if (ev_from_arg) ev[0] = ev0;
    }
    const EventDesc E = ev_from_arg ? ev0 : ev[blockIdx.y];
    const int tid = blockIdx.x * kBlock + threadIdx.x;
    const int stride = gridDim.x * kBlock;
    const long long total = static_cast<long long>(E.n) * d;
    const float *Xe = E.pts;
    float mn[kMaxAxes] = {INFINITY, INFINITY, INFINITY, INFINITY};
    float mx[kMaxAxes] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    // A thread's elements (float4 groups, or single ones) are a whole number of rows
    // apart, so that it sees the same columns every time and needs no look at them per
    // element: a minimum, a maximum and a comparison each (with the column tracked and
    // compared per element the pass was bound by its instructions: 67 us against 52 on a
    // batch of 5.6M 8-D points, 8.9 against 5.5 on 300k 12-D and 8.2 against 4.3 on 47k
    // 10-D ones, whose rows are read one float at a time).  Several loads are in flight
    // per thread, issued together also for the last, partial round (the grid gives most
    // threads exactly four).
    if (vec4) {
        const float4 *X4 = reinterpret_cast<const float4 *>(Xe);
        const long long nv = total / 4;
        const int groups = d / 4;
        const long long step = static_cast<long long>(stride / groups) * groups;
        BoundsAcc<4> acc;
        for (long long v = tid < step ? tid : nv; v < nv; v += 4 * step) {
            float4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // Past the end the thread's own first group is read again.
                const long long w = v + u * step;
                x[u] = X4[w < nv ? w : v];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc.add(0, x[u].x);
                acc.add(1, x[u].y);
                acc.add(2, x[u].z);
                acc.add(3, x[u].w);
            }
        }
        bad = acc.bad();
        const int col = 4 * (tid % groups);
#pragma unroll
        for (int p = 0; p < kMaxAxes; ++p)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (col + k == dd.c[p]) {
                    mn[p] = acc.mn[k];
                    mx[p] = acc.mx[k];
                }
    } else {
        const long long step = static_cast<long long>(stride / d) * d;
        BoundsAcc<1> acc;
        for (long long e = tid < step ? tid : total; e < total; e += 8 * step) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const long long w = e + u * step;
                x[u] = Xe[w < total ? w : e];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) acc.add(0, x[u]);
        }
        bad = acc.bad();
        const int col = tid % d;
#pragma unroll
        for (int p = 0; p < kMaxAxes; ++p)
            if (col == dd.c[p]) {
                mn[p] = acc.mn[0];
                mx[p] = acc.mx[0];
            }
    }
#pragma unroll
    for (int p = 0; p < kMaxAxes; ++p) {
        mn[p] = wave_min(mn[p]);
        mx[p] = wave_max(mx[p]);
    }
    bad = wave_any(bad);
    __shared__ BoundsPartial sp[kWaves];
    if (lane_id() == 0) {
        BoundsPartial &p = sp[wave_id()];
        for (int q = 0; q < kMaxAxes; ++q) {
            p.mn[q] = mn[q];
            p.mx[q] = mx[q];
        }
        p.nonfinite = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        BoundsPartial out = sp[0];
        for (int w = 1; w < kWaves; ++w) {
            for (int p = 0; p < kMaxAxes; ++p) {
                out.mn[p] = fminf(out.mn[p], sp[w].mn[p]);
                out.mx[p] = fmaxf(out.mx[p], sp[w].mx[p]);
            }
            out.nonfinite |= sp[w].nonfinite;
        }
        out.pad = 0;
        part[static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x] = out;
    }
}

// ------------------------------------------------------------------- keys

// Wave 0 of a block folds the bounds partials and derives the grid, lane p axis p.
// Every block derives the same plan from the same partials (min/max are exact).
// Axes from `axes` on are not binned: one cell each.
__device__ void derive_plan(const BoundsPartial *__restrict__ part, int nparts, float r,
                            int cell_div, int axes, int cells_max, int n, int tile_points, Plan *out) {
    float mn[kMaxAxes] = {INFINITY, INFINITY, INFINITY, INFINITY};
    float mx[kMaxAxes] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    // Every lane loads its (at most kBoundsBlocks / 64) partials before folding them.
    constexpr int kPartsPerLane = kBoundsBlocks / 64;
    BoundsPartial pb[kPartsPerLane];
#pragma unroll
    for (int u = 0; u < kPartsPerLane; ++u) {
        const int b = lane_id() + 64 * u;
        if (b < nparts) pb[u] = part[b];
    }
#pragma unroll
    for (int u = 0; u < kPartsPerLane; ++u) {
        if (lane_id() + 64 * u >= nparts) continue;
        for (int p = 0; p < kMaxAxes; ++p) {
            mn[p] = fminf(mn[p], pb[u].mn[p]);
            mx[p] = fmaxf(mx[p], pb[u].mx[p]);
        }
        bad |= pb[u].nonfinite;
    }
#pragma unroll
    for (int p = 0; p < kMaxAxes; ++p) {
        mn[p] = wave_min(mn[p]);
        mx[p] = wave_max(mx[p]);
    }
    bad = wave_any(bad);
    // Cell edge r (1 + 2^-10) / cell_div.  A pair that passes the float32 test has
    // |x_p - y_p| < r exactly along every coordinate (partial sums never exceed D,
    // rounding is monotone); the 2^-10 margin absorbs the float32 rounding of the
    // key computation (at most 3 * 2^-24 * G cells per point, G <= 1024), so such
    // a pair lands at most cell_div cells apart along every binned axis.  Larger
    // cells only keep such pairs closer.
    const float cbase = (r * 1.0009765625f) / static_cast<float>(cell_div);
    const int axis_max = axes == 4 ? kGridAxisMax4 : kGridAxisMax3;
    const float axis_soft = axes == 4 ? 250.0f : 1000.0f;
    const int p = lane_id() & (kMaxAxes - 1);
    float lo = mn[0], hi = mx[0];
#pragma unroll
    for (int k = 1; k < kMaxAxes; ++k) {
        lo = p == k ? mn[k] : lo;
        hi = p == k ? mx[k] : hi;
    }
    // An axis whose extent is not a finite float (no points, or max - min
    // overflowing), or that is not binned, gets a single cell: inv_c = 0 puts
    // every point in cell 0.
    const float ext = hi - lo;
    bool single = p >= axes || !(ext >= 0.0f && ext <= FLT_MAX);
    if (!(lo <= hi)) lo = 0.0f;
    float c = cbase;
    if (!single && ext / c > axis_soft) c = ext / axis_soft;
    // Grow the cells until the grid fits cells_max (bounded: after 128 rounds of
    // x1.25 every finite extent spans one cell).
    int G = 1;
    long long total = 1;
    for (int round = 0;; ++round) {
        float g = single ? 1.0f : floorf(ext / c) + 1.0f;
        if (!(g <= static_cast<float>(axis_max))) g = static_cast<float>(axis_max);
        if (!(g >= 1.0f)) g = 1.0f;
        G = static_cast<int>(g);
        total = static_cast<long long>(__builtin_amdgcn_readlane(G, 0)) * __builtin_amdgcn_readlane(G, 1) *
                __builtin_amdgcn_readlane(G, 2) * __builtin_amdgcn_readlane(G, 3);
        if (total <= cells_max) break;
        if (round >= 128) single = true;
        else c *= 1.25f;
    }
    if (lane_id() < kMaxAxes) {
        out->lo[p] = p < axes ? lo : 0.0f;
        out->c[p] = single ? INFINITY : c;
        out->inv_c[p] = single ? 0.0f : 1.0f / c;
        out->G[p] = G;
    }
    if (lane_id() != 0) return;
    out->n_cells = static_cast<int>(total);
    out->reach = cell_div;
    out->abort = bad;
    out->axes = axes;
    if (tile_points == 0) return;  // not binned through tiles
    // Cells per tile of the tile pass: the power of two that gives a tile at most
    // tile_points points on average.
    int shift = 0;
    while (shift < kTileShiftMax &&
           static_cast<long long>(n) << (shift + 1) <= static_cast<long long>(out->n_cells) * tile_points)
        ++shift;
    out->tile_shift = shift;
    out->n_tiles = (out->n_cells + (1 << shift) - 1) >> shift;
}

// Clamping is monotone and moves no coordinate by more than the clamp, so two
// points that are at most R cells apart stay at most R cells apart.
__device__ __forceinline__ int cell_coord(float x, float lo, float inv_c, int G) {
    float q = floorf((x - lo) * inv_c);
    q = fmaxf(q, 0.0f);  // also maps NaN to 0
    q = fminf(q, static_cast<float>(G - 1));
    return static_cast<int>(q);
}

// Cell coordinates of a point pack into one word (cell_bits per axis); the cell
// key orders cells with axis 0 fastest, so the cells along axis 0 around a cell
// are contiguous in cell order.
__device__ __forceinline__ unsigned int pack_cell(const int (&u)[kMaxAxes], int axes) {
    const int b = cell_bits(axes);
    return static_cast<unsigned int>(u[0]) | static_cast<unsigned int>(u[1]) << b |
           static_cast<unsigned int>(u[2]) << (2 * b) | static_cast<unsigned int>(u[3]) << (3 * b);
}

__device__ __forceinline__ void unpack_cell(unsigned int pc, int axes, int (&u)[kMaxAxes]) {
    const int b = cell_bits(axes);
    const unsigned int m = (1u << b) - 1u;
#pragma unroll
    for (int p = 0; p < kMaxAxes; ++p) u[p] = static_cast<int>((pc >> (p * b)) & m);
}

__device__ __forceinline__ unsigned int cell_key(const int (&u)[kMaxAxes], const Plan &P) {
    return static_cast<unsigned int>(((u[3] * P.G[2] + u[2]) * P.G[1] + u[1]) * P.G[0] + u[0]);
}

constexpr int kMaxCellTiles = ((1 << 24) + kScanTile - 1) / kScanTile + 2;

// Grid (blocks, n_events) of kKeysBlock threads: block 0 of event e derives and
// stores its plan; every block computes the cells of kKeysBlock x kKeysPer of the
// event's rows.  Two points per thread halve the blocks, and with them the
// blocks' atomic adds to each tile total, which pays for large events.
__global__ __launch_bounds__(kKeysBlock) void k_keys(int d, Dims dd, int axes,
                                                     float r, int cell_div,
                                                     const EventDesc *__restrict__ ev, EventDesc ev0, int ev_from_arg,
                                                     const BoundsPartial *__restrict__ part, int nparts,
                                                     Plan *__restrict__ plans, Counters *__restrict__ ctr,
                                                     unsigned int *__restrict__ pcell,
                                                     unsigned int *__restrict__ rank,
                                                     unsigned int *__restrict__ cell_count,
                                                     unsigned long long *__restrict__ sums_cells) {
    __shared__ Plan P;
    // Per scan tile: points (low word) and newly occupied cells (high word).
    __shared__ unsigned long long tile_count[kMaxCellTiles];
    const int e = blockIdx.y;
    const EventDesc E = ev_from_arg ? ev0 : ev[e];  // one event: no load before the points'
    constexpr int kSpan = kKeysSpan;
    if (blockIdx.x != 0 && static_cast<long long>(blockIdx.x) * kSpan >= E.n) return;
    // kKeysPer points per thread, kKeysBlock apart; their binned coordinates are
    // loaded before the plan is derived so that the two latencies overlap.
    float x[kKeysPer][kMaxAxes];
#pragma unroll
    for (int m = 0; m < kKeysPer; ++m) {
        const int i = blockIdx.x * kSpan + m * kKeysBlock + threadIdx.x;
#pragma unroll
        for (int p = 0; p < kMaxAxes; ++p) x[m][p] = 0.0f;
        if (i < E.n) {
            const float *row = E.pts + static_cast<size_t>(i) * d;
#pragma unroll
            for (int p = 0; p < kMaxAxes; ++p)
                if (p < axes) x[m][p] = row[dd.c[p]];
        }
    }
    if (wave_id() == 0)
        derive_plan(part + static_cast<size_t>(e) * nparts, nparts, r, cell_div, axes, E.cells_max, E.n, 0, &P);
    const int tile_end = static_cast<int>((E.cell0 + E.cells_max - 1) / kScanTile);
    const int ntiles = tile_end - E.tile0 + 1;
    for (int t = threadIdx.x; t < ntiles; t += kKeysBlock) tile_count[t] = 0ull;
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        plans[e] = P;
        if (P.abort) atomicOr(&ctr->abort, 1u);
    }
    if (P.abort) return;
    unsigned int k[kKeysPer], rk[kKeysPer];
#pragma unroll
    for (int m = 0; m < kKeysPer; ++m) {
        const int i = blockIdx.x * kSpan + m * kKeysBlock + threadIdx.x;
        if (i >= E.n) continue;
        const long long gi = E.row0 + i;
        int u[kMaxAxes];
#pragma unroll
        for (int p = 0; p < kMaxAxes; ++p) u[p] = cell_coord(x[m][p], P.lo[p], P.inv_c[p], P.G[p]);
        k[m] = static_cast<unsigned int>(E.cell0) + cell_key(u, P);
        pcell[gi] = pack_cell(u, axes);
        rk[m] = atomicAdd(&cell_count[k[m]], 1u);
    }
#pragma unroll
    for (int m = 0; m < kKeysPer; ++m) {
        const int i = blockIdx.x * kSpan + m * kKeysBlock + threadIdx.x;
        if (i >= E.n) continue;
        rank[E.row0 + i] = rk[m];
        // The first point of a cell (rank 0) also counts the cell as occupied.
        atomicAdd(&tile_count[k[m] / kScanTile - E.tile0], rk[m] == 0u ? (1ull << 32) | 1ull : 1ull);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < ntiles; t += kKeysBlock)
        if (tile_count[t]) atomicAdd(&sums_cells[E.tile0 + t], tile_count[t]);
}

// ------------------------------------------------------------------- scans

// Workgroups of the search before those of XCD x (0..8): workgroups are dealt to the 8
// XCDs round-robin, and each XCD works on a contiguous share of the pieces.
__device__ __forceinline__ unsigned int xcd_first_block(unsigned int x, unsigned int blocks) {
    return x * (blocks / 8u) + min(x, blocks % 8u);
}

// The queries with long lists are queued per XCD, in the part of long_slots that
// belongs to the XCD's rows: lists that a wave of the placement pass can collect from
// the front, larger ones from the back.  With one counter for all of them the search of
// an event with many long lists waited for its atomics, one per wave that writes lists
// out: 87 us against 30 for 60,000 points with some 45 neighbours each, 45 against 22
// for 20,000 in denser ones, 32.4 against 27.5 for a 120k-point event where 2% of the
// lists are long.  The lanes of a wave add one each to the same address; the compiler makes
// one atomic of theirs, by the first lane, of as many as they are (a test looks for it).
constexpr int kLongCount = 1, kHugeCount = 2, kExtCount = 3;  // words of an XCD's line of counters
__device__ __forceinline__ unsigned int *long_counter(unsigned int *claims, unsigned int xcd, int which) {
    return claims + xcd * kClaimStride + which;
}

// floor(a / b) for a < 2^52, b > 0: the quotient rounded in double is within one
// of the exact, and integer products settle it.
__device__ __forceinline__ unsigned long long floor_div(unsigned long long a, unsigned long long b) {
    unsigned long long f = static_cast<unsigned long long>(static_cast<double>(a) / static_cast<double>(b));
    if (f * b > a) --f;
    if ((f + 1) * b <= a) ++f;
    return f;
}

// cell_start[c] = points in cells [0, c) for c in [0, cells]; sums[t] holds tile
// t's points (low word) and occupied cells (high word).  The tile's counts are
// requested before the totals of the tiles before it are summed, so that the two
// round trips overlap.
//
// The same pass divides the queries into the search's n_waves pieces by work
// rather than by count: a cell weighs its points plus kTileWeight if it has any
// (a tile's fixed cost, in queries), the cells in order span weights [0, W), and
// wave k starts at weight floor(k W / n_waves), which falls in one cell; the wave
// starts there at the query that many weight units past the cell's fixed cost
// (at its first query if it falls within the cost), so a dense cell can still be
// split among waves.  wave_start[k] is that sorted row; wave_start[n_waves] =
// rows.  The pieces that start in a tile are taken one per thread, each finding its
// cell by bisection over the tile's weights in LDS.  (Walked cell by cell in the thread
// that holds the cells, every lane waits for the fullest cell of its wave, 16 times
// over: 51 us against 4.6 for 2,000 points, 23 against 6.8 for 20,000 in crowded cells,
// 5.5 against 5.2 for 120,000 in sparse ones.)
__global__ __launch_bounds__(kBlock) void k_scan_cells(const unsigned int *__restrict__ in, long long len,
                                                       const unsigned long long *__restrict__ sums, int tiles,
                                                       unsigned int *__restrict__ out,
                                                       unsigned int *__restrict__ wave_start, int n_waves,
                                                       long long rows, unsigned int *__restrict__ claims) {
    __shared__ unsigned long long red[4 * kWaves];
    __shared__ __align__(16) unsigned int cell_w[kScanTile], cell_c[kScanTile];
    __shared__ unsigned int tile_w;
    const long long base = static_cast<long long>(blockIdx.x) * kScanTile;
    if (base > len) return;
    constexpr int kPer = kScanTile / kBlock;
    static_assert(kPer % 4 == 0, "a thread's counts are read as 16-byte groups");
    // A thread's kPer counts are consecutive (16-byte aligned: the tile and the
    // workspace arrays are): whole groups are read as uint4, the last thread's
    // partial group one by one.
    unsigned int v[kPer];
    const long long first = base + static_cast<long long>(threadIdx.x) * kPer;
    if (first + kPer <= len) {
        const uint4 *src = reinterpret_cast<const uint4 *>(in + first);
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j) {
            const uint4 g = src[j];
            v[4 * j] = g.x;
            v[4 * j + 1] = g.y;
            v[4 * j + 2] = g.z;
            v[4 * j + 3] = g.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kPer; ++j) v[j] = first + j < len ? in[first + j] : 0u;
    }
    // Points and weight of the tiles before this one, and the weight of them all.
    unsigned long long c_before = 0, w_before = 0, w_all = 0;
    for (int t = threadIdx.x; t < tiles; t += kBlock) {
        const unsigned long long x = sums[t];
        const unsigned long long w = (x & 0xffffffffull) + kTileWeight * (x >> 32);
        w_all += w;
        if (t < static_cast<int>(blockIdx.x)) {
            c_before += x & 0xffffffffull;
            w_before += w;
        }
    }
    // This thread's points (low word) and weight (high word); a block's totals of
    // either stay below 2^32, so the packed scan carries nothing between them.
    unsigned long long mine = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        mine += (static_cast<unsigned long long>(v[j] + (v[j] ? kTileWeight : 0u)) << 32) | v[j];
    c_before = wave_sum(c_before);
    w_before = wave_sum(w_before);
    w_all = wave_sum(w_all);
    const unsigned long long inc = wave_inclusive_scan(mine);
    if (lane_id() == 63) {
        red[wave_id()] = c_before;
        red[kWaves + wave_id()] = w_before;
        red[2 * kWaves + wave_id()] = w_all;
        red[3 * kWaves + wave_id()] = inc;
    }
    __syncthreads();
    unsigned long long cb = 0, wb = 0, W = 0, pre = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        cb += red[w];
        wb += red[kWaves + w];
        W += red[2 * kWaves + w];
        pre += w < wave_id() ? red[3 * kWaves + w] : 0ull;
    }
    pre += inc - mine;
    // The tile's counts and weights before each cell (relative to the tile's first).
    unsigned int run_c = static_cast<unsigned int>(pre), run_w = static_cast<unsigned int>(pre >> 32);
    const unsigned int first_row = static_cast<unsigned int>(cb);  // rows stay below 2^31
    unsigned int starts[kPer], weights[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        starts[j] = first_row + run_c;
        weights[j] = run_w;
        run_c += v[j];
        run_w += v[j] + (v[j] ? kTileWeight : 0u);
    }
    // cell_start has len + 1 entries: whole groups as uint4, the rest one by one.
    if (first + kPer <= len + 1) {
        uint4 *dst = reinterpret_cast<uint4 *>(out + first);
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j)
            dst[j] = make_uint4(starts[4 * j], starts[4 * j + 1], starts[4 * j + 2], starts[4 * j + 3]);
    } else {
#pragma unroll
        for (int j = 0; j < kPer; ++j)
            if (first + j <= len) out[first + j] = starts[j];
    }
    {
        uint4 *ws = reinterpret_cast<uint4 *>(cell_w + threadIdx.x * kPer);
        uint4 *cs = reinterpret_cast<uint4 *>(cell_c + threadIdx.x * kPer);
#pragma unroll
        for (int j = 0; j < kPer / 4; ++j) {
            ws[j] = make_uint4(weights[4 * j], weights[4 * j + 1], weights[4 * j + 2], weights[4 * j + 3]);
            cs[j] = make_uint4(starts[4 * j], starts[4 * j + 1], starts[4 * j + 2], starts[4 * j + 3]);
        }
        if (threadIdx.x == kBlock - 1) tile_w = run_w;
    }
    __syncthreads();
    // Pieces k with B_k = floor(k W / n) in the tile's weights [wb, wb + tile_w): those
    // with k W >= wb n and k W < (wb + tile_w) n.
    if (W && tile_w) {
        const unsigned long long nw = static_cast<unsigned long long>(n_waves);
        unsigned long long k0 = floor_div(wb * nw + W - 1, W);
        const unsigned long long k1 = floor_div((wb + tile_w) * nw + W - 1, W);
        if (k0 == 0) k0 = 1;  // wave 0 starts at row 0
        for (unsigned long long k = k0 + threadIdx.x; k < k1 && k < nw; k += kBlock) {
            const unsigned int at = static_cast<unsigned int>(floor_div(k * W, nw) - wb);
            int lo = 0, hi = kScanTile - 1;  // the last cell that starts at or before it
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (cell_w[mid] <= at) lo = mid;
                else hi = mid - 1;
            }
            const unsigned int past = at - cell_w[lo];
            wave_start[k] = cell_c[lo] + (past > kTileWeight ? past - kTileWeight : 0u);
        }
    }
    if (blockIdx.x == 0) {
        static_assert(kExtCount < kClaimStride, "a line per XCD");
        if (threadIdx.x < 8) {
            *long_counter(claims, threadIdx.x, kLongCount) = 0u;
            *long_counter(claims, threadIdx.x, kHugeCount) = 0u;
            *long_counter(claims, threadIdx.x, kExtCount) = 0u;
        }
        if (W == 0) {  // no rows: every share is empty
            for (int t = threadIdx.x; t <= n_waves; t += kBlock) wave_start[t] = 0u;
        } else if (threadIdx.x == 0) {
            wave_start[0] = 0u;
            wave_start[n_waves] = static_cast<unsigned int>(rows);
        }
    }
}

// ----------------------------------------------------------------- scatter

// Grid (blocks, n_events): block (b, e) copies a share of event e's rows.
template <int DP>
__global__ __launch_bounds__(kBlock) void k_scatter(int d, int vec4, const EventDesc *__restrict__ ev,
                                                    EventDesc ev0, int ev_from_arg,
                                                    const Plan *__restrict__ plans,
                                                    const unsigned int *__restrict__ pcell,
                                                    const unsigned int *__restrict__ rank,
                                                    const unsigned int *__restrict__ cell_start,
                                                    const Counters *__restrict__ ctr,
                                                    float *__restrict__ sorted, long long rows,
                                                    unsigned int *__restrict__ sorted_id) {
    // The point's packed cell, rank and row are requested before the abort flag is
    // known (they are in bounds whatever it says); the cell start, whose index needs
    // a valid plan, only when it is clear.
    const bool abort = ctr->abort != 0;
    const EventDesc E = ev_from_arg ? ev0 : ev[blockIdx.y];
    const Plan P = plans[blockIdx.y];
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < E.n; i += gridDim.x * kBlock) {
        const long long gi = E.row0 + i;
        const unsigned int pc = pcell[gi];
        const unsigned int rk = rank[gi];
        float row[DP];
        if (vec4) {
            const float4 *src = reinterpret_cast<const float4 *>(E.pts + static_cast<size_t>(i) * d);
#pragma unroll
            for (int k = 0; k < DP / 4; ++k) {
                float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (4 * k < d) v = src[k];
                row[4 * k] = v.x;
                row[4 * k + 1] = v.y;
                row[4 * k + 2] = v.z;
                row[4 * k + 3] = v.w;
            }
        } else {
            const float *src = E.pts + static_cast<size_t>(i) * d;
#pragma unroll
            for (int k = 0; k < DP; ++k) row[k] = k < d ? src[k] : 0.0f;
        }
        if (abort) return;
        int u[kMaxAxes];
        unpack_cell(pc, P.axes, u);
        const unsigned int slot = cell_start[static_cast<unsigned int>(E.cell0) + cell_key(u, P)] + rk;
        SortedRows<DP>::store(sorted, rows, slot, row);
        // The original row and the packed cell of a sorted row sit side by side, so
        // the scattered write is one 8-byte store instead of two 4-byte ones.
        reinterpret_cast<uint2 *>(sorted_id)[slot] = make_uint2(static_cast<unsigned int>(gi), pc);
    }
}

// --------------------------------------------------- binning through tiles in LDS

// Events of up to kBinMaxRows rows are sorted into cells without an atomic on global
// memory per point: k_bin sorts each share of points by tile (a run of cells) in LDS, and
// k_tiles gathers one tile's points from all shares, counts and orders them by cell in
// LDS and writes rows, cell starts and search shares.  By atomics (k_keys, k_scan_cells,
// k_scatter: events beyond what the tiles' tables hold, see kBinMaxRows) every point takes
// a returning atomic beyond its XCD's L2 and its row is written to a place that shares its
// lines with rows of other XCDs.  One 120k-point event: 13.7, 5.1 and 6.9 us by atomics,
// 8.5 and 10.5 through tiles; 300k 12-D points: 22.0, 5.6 and 14.7 against 10.1 and 19.3; a
// batch of 64 events (5.6M points): 240, 34 and 217 against 92 and 198, where k_tiles is
// bound by memory (1.1 GB at 5.4 TB/s: a line of points holds the rows of several tiles
// and is fetched for each; giving each event's tiles to one XCD took 235 us, the XCDs'
// shares being uneven).

// Exclusive prefixes over the block in thread order of two values, and the block's totals
// of both, for a block of WAVES waves, with one barrier (scratch belongs to this call).
template <int WAVES>
__device__ __forceinline__ uint2 block_prefix2(uint2 v, uint2 *scratch, uint2 &total) {
    const uint2 inc = make_uint2(wave_inclusive_scan(v.x), wave_inclusive_scan(v.y));
    if (lane_id() == 63) scratch[wave_id()] = inc;
    __syncthreads();
    uint2 before = make_uint2(0u, 0u), all = make_uint2(0u, 0u);
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const uint2 x = scratch[w];
        before.x += w < wave_id() ? x.x : 0u;
        before.y += w < wave_id() ? x.y : 0u;
        all.x += x.x;
        all.y += x.y;
    }
    total = all;
    return make_uint2(before.x + inc.x - v.x, before.y + inc.y - v.y);
}

__device__ __forceinline__ int bin_shares(int n, int span) { return (n + span - 1) / span; }

// The event, and the share or tile of it, that a block works on.  Grids are (blocks of
// the largest event, n_events) as a rule.  Where most of those blocks would find nothing
// to do (a large event among many small ones) the grid has one dimension, in which event
// e's blocks begin at blocks_before: one for every `rows` rows before it, rounded down,
// and `extra` for every event before it.
__host__ __device__ __forceinline__ long long blocks_before(long long row0, long long e, int rows, int extra) {
    return static_cast<unsigned int>(row0) / static_cast<unsigned int>(rows) + e * extra;  // rows below 2^31
}
__device__ __forceinline__ int2 event_block(const EventDesc *__restrict__ ev, int flat_events, int rows, int extra) {
    if (flat_events == 0) return make_int2(blockIdx.y, blockIdx.x);
    int lo = 0, hi = flat_events - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (blocks_before(ev[mid].row0, mid, rows, extra) <= static_cast<long long>(blockIdx.x)) lo = mid;
        else hi = mid - 1;
    }
    return make_int2(lo, static_cast<int>(blockIdx.x - blocks_before(ev[lo].row0, lo, rows, extra)));
}
// Blocks of k_tiles in a one-dimensional grid: tile_blocks(n) is at most one for every
// tile_block_rows rows, and these more (an odd number, as below).
constexpr int kTilesExtra = 11;
constexpr int tile_block_rows(int tile_points) { return 32 * tile_points / 65; }

// Grid (shares, n_events): block (b, e) takes rows [b span, (b + 1) span) of event e.  It
// writes each row's number and packed cell in the order of the rows' tiles to the same
// range of ents, and where each tile starts in the share to row b of the event's table
// (n_tiles + 1 entries, in the event's part of the histogram's memory).  A tile of which
// the share holds many points gets them added to its count (crowd_reported).
template <int kPer>
__global__ __launch_bounds__(kKeysBlock) void k_bin(int d, Dims dd, int axes, float r, int cell_div,
                                                    int tile_points, const EventDesc *__restrict__ ev, EventDesc ev0, int ev_from_arg,
                                                    int flat_events,
                                                    const BoundsPartial *__restrict__ part, int nparts,
                                                    Plan *__restrict__ plans, Counters *__restrict__ ctr,
                                                    uint2 *__restrict__ ents, unsigned short *__restrict__ table,
                                                    unsigned int *__restrict__ crowd,
                                                    unsigned long long *__restrict__ crowd_sum) {
    __shared__ Plan P;
    __shared__ unsigned int start[kBinMaxTiles];  // rows per tile, then where the tile starts
    __shared__ uint2 scratch[kKeysBlock / 64];
    constexpr int kSpan = kKeysBlock * kPer;
    const int2 at = event_block(ev, flat_events, kSpan, 1);
    const int e = at.x, share = at.y;
    const EventDesc E = ev_from_arg ? ev0 : ev[e];
    if (share != 0 && static_cast<long long>(share) * kSpan >= E.n) return;
    // The binned coordinates are loaded before the plan is derived so that the two
    // latencies overlap.
    float x[kPer][kMaxAxes];
#pragma unroll
    for (int m = 0; m < kPer; ++m) {
        const int i = share * kSpan + m * kKeysBlock + threadIdx.x;
#pragma unroll
        for (int p = 0; p < kMaxAxes; ++p) x[m][p] = 0.0f;
        if (i < E.n) {
            const float *row = E.pts + static_cast<size_t>(i) * d;
#pragma unroll
            for (int p = 0; p < kMaxAxes; ++p)
                if (p < axes) x[m][p] = row[dd.c[p]];
        }
    }
    if (wave_id() == 0)
        derive_plan(part + static_cast<size_t>(e) * nparts, nparts, r, cell_div, axes, E.cells_max, E.n, tile_points,
                    &P);
    for (int t = threadIdx.x; t < kBinMaxTiles; t += kKeysBlock) start[t] = 0u;
    __syncthreads();
    if (share == 0 && threadIdx.x == 0) {
        plans[e] = P;
        if (P.abort) atomicOr(&ctr->abort, 1u);
    }
    if (P.abort) return;
    const int n_tiles = P.n_tiles;
    unsigned int tile[kPer], rank[kPer], pc[kPer];
#pragma unroll
    for (int m = 0; m < kPer; ++m) {
        const int i = share * kSpan + m * kKeysBlock + threadIdx.x;
        if (i >= E.n) continue;
        int u[kMaxAxes];
#pragma unroll
        for (int p = 0; p < kMaxAxes; ++p) u[p] = cell_coord(x[m][p], P.lo[p], P.inv_c[p], P.G[p]);
        pc[m] = pack_cell(u, axes);
        tile[m] = cell_key(u, P) >> P.tile_shift;
        rank[m] = atomicAdd(&start[tile[m]], 1u);
    }
    __syncthreads();
    // Four consecutive tiles per thread.
    static_assert(kBinMaxTiles == 4 * kKeysBlock, "four tiles per thread");
    uint4 c = *reinterpret_cast<const uint4 *>(start + 4 * threadIdx.x);
    const unsigned int held[4] = {c.x, c.y, c.z, c.w};
    uint2 all;
    const unsigned int pre = block_prefix2<kKeysBlock / 64>(make_uint2(c.x + c.y + c.z + c.w, 0u), scratch, all).x;
    c = make_uint4(pre, pre + c.x, pre + c.x + c.y, pre + c.x + c.y + c.z);
    *reinterpret_cast<uint4 *>(start + 4 * threadIdx.x) = c;
    __syncthreads();
    unsigned short *row = table + 2 * E.cell0 + static_cast<size_t>(share) * (n_tiles + 1);
    for (int t = threadIdx.x; t <= n_tiles; t += kKeysBlock)
        row[t] = static_cast<unsigned short>(t < n_tiles ? start[t] : all.x);
#pragma unroll
    for (int m = 0; m < kPer; ++m) {
        const int i = share * kSpan + m * kKeysBlock + threadIdx.x;
        if (i >= E.n) continue;
        ents[E.row0 + static_cast<long long>(share) * kSpan + start[tile[m]] + rank[m]] =
            make_uint2(static_cast<unsigned int>(i), pc[m]);
    }
    const int shares = bin_shares(E.n, kSpan);
    const bool many = E.n >= crowd_points(tile_points, shares) &&
                      crowd_reported(max(max(held[0], held[1]), max(held[2], held[3])), tile_points, shares);
    if (__builtin_amdgcn_ballot_w64(many) != 0ull) {
        unsigned int sum = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (many && crowd_reported(held[k], tile_points, shares)) {
                atomicAdd(crowd + crowd_at(E.row0, tile_points) + 4 * threadIdx.x + k, held[k]);
                sum += held[k];
            }
        sum = wave_sum(sum);
        if (lane_id() == 0) atomicAdd(crowd_sum + e, static_cast<unsigned long long>(sum));
    }
}

// Grid (tiles, n_events): block (t, e) finishes tile t of event e: its points' cells
// counted in LDS, the cells' first sorted rows, the search's pieces that start in the
// tile, then the rows themselves, copied into cell order and zero-padded to DP.
//
// The pieces are dealt to the tiles by rows (a tile of some hundred points has about the
// same mix of cells as the next) and cut inside a tile by work: a cell weighs its points
// plus kTileWeight if it has any.  Piece k ideally starts at row k rows / n_pieces; in
// its tile it starts at the same share of the tile's weight, at the query that many
// weight units past its cell's fixed cost (at the cell's first query if it falls within
// the cost).
//
// A crowded tile (crowd_points) is worked off in parts, each the points of a run of shares:
// part 0 by the tile's own block, the others by blocks past the event's tiles, which find
// theirs by a prefix over the tiles' counts.  Every part counts all of the tile's points,
// those of earlier parts apart, so that it knows where its own go in each cell.
template <int DP>
__global__ __launch_bounds__(kTilesBlock) void k_tiles(int d, int vec4, int span, const EventDesc *__restrict__ ev,
                                                       EventDesc ev0, int ev_from_arg, int flat_events,
                                                       int tile_points,
                                                       const Plan *__restrict__ plans,
                                                       const uint2 *__restrict__ ents,
                                                       const unsigned short *__restrict__ table,
                                                       const unsigned int *__restrict__ crowd,
                                                       const unsigned long long *__restrict__ crowd_sum,
                                                       unsigned int *__restrict__ cell_start,
                                                       float *__restrict__ sorted,
                                                       unsigned int *__restrict__ sorted_id,
                                                       unsigned int *__restrict__ wave_start, int n_pieces,
                                                       long long rows, unsigned int *__restrict__ claims) {
    constexpr int kTWaves = kTilesBlock / 64;
    constexpr int kCells = 1 << kTileShiftMax;
    __shared__ __align__(16) unsigned int cursor[kCells];  // points per cell, then where the cell starts in the tile
    __shared__ __align__(16) unsigned int weight[kCells];  // weight before the cell in the tile (a part's later points first)
    __shared__ unsigned int seg_pre[kBinMaxShares + 1];  // points of the tile in the shares before (past the last: all)
    __shared__ unsigned int seg_from[kBinMaxShares];  // where the share's points of the tile lie in ents
    __shared__ uint2 scratch[3][kTWaves];
    __shared__ int2 my_part;
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        static_assert(kExtCount < kClaimStride, "a line per XCD");
        if (threadIdx.x < 8) {
            *long_counter(claims, threadIdx.x, kLongCount) = 0u;
            *long_counter(claims, threadIdx.x, kHugeCount) = 0u;
            *long_counter(claims, threadIdx.x, kExtCount) = 0u;
        }
        if (threadIdx.x == 0) wave_start[n_pieces] = static_cast<unsigned int>(rows);
    }
    const int2 which = event_block(ev, flat_events, tile_block_rows(tile_points), kTilesExtra);
    int t = which.y;
    const EventDesc E = ev_from_arg ? ev0 : ev[which.x];
    const Plan P = plans[which.x];
    // Points of crowded tiles (no tile is where crowd_sum is null): a vector load, so that only
    // the blocks that use it at once wait.
    unsigned int crowded_v = 0u;
    if (crowd_sum)
        crowded_v = static_cast<unsigned int>(
            __hip_atomic_load(crowd_sum + which.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT));
    if (P.abort || E.n == 0) return;
    const int shares = bin_shares(E.n, span);
    const unsigned int *__restrict__ counts = crowd + crowd_at(E.row0, tile_points);
    // Workgroups of tile k beside its own.
    auto more_of = [&](int k, int shift) -> unsigned int {
        const unsigned int counted = counts[k];
        return counted >= static_cast<unsigned int>(crowd_points(tile_points, shares)) ? counted >> shift : 0u;
    };
    int part = 0, parts = 1;
    if (t >= P.n_tiles) {
        // The x-th of the parts past the first of the event's tiles.
        if (!crowd_sum || E.n < crowd_least(tile_points)) return;
        const unsigned int x = static_cast<unsigned int>(t - P.n_tiles), crowded = uniform(crowded_v);
        if (x >= crowded >> (__builtin_ctz(tile_points) + 2)) return;
        const int shift = crowd_shift(crowded, E.n, P.n_tiles, tile_points);
        const int per = (P.n_tiles + kTilesBlock - 1) / kTilesBlock;
        const int t0 = min(static_cast<int>(threadIdx.x) * per, P.n_tiles), t1 = min(t0 + per, P.n_tiles);
        unsigned int more = 0;
        for (int k = t0; k < t1; ++k) more += more_of(k, shift);
        uint2 all;
        unsigned int before = block_prefix2<kTWaves>(make_uint2(more, 0u), scratch[2], all).x;
        if (x >= all.x) return;
        if (before <= x && x < before + more) {
            for (int k = t0; k < t1; ++k) {
                const unsigned int m = more_of(k, shift);
                if (before <= x && x < before + m) my_part = make_int2(k, static_cast<int>(x - before) + 1);
                before += m;
            }
        }
        __syncthreads();
        t = static_cast<int>(uniform(static_cast<unsigned int>(my_part.x)));
        part = static_cast<int>(uniform(static_cast<unsigned int>(my_part.y)));
    }
    // The tile's segment of every share (one share per thread).
    static_assert(kBinMaxShares == kTilesBlock, "one share per thread");
    unsigned int from = 0, len = 0;
    if (static_cast<int>(threadIdx.x) < shares) {
        const unsigned short *row = table + 2 * E.cell0 + static_cast<size_t>(threadIdx.x) * (P.n_tiles + 1) + t;
        from = row[0];
        len = row[1] - from;
    }
    const unsigned int key0 = static_cast<unsigned int>(t) << P.tile_shift;  // the tile's first cell
    const int cells = min(1 << P.tile_shift, P.n_cells - static_cast<int>(key0));
    for (int c = threadIdx.x; c < cells; c += kTilesBlock) cursor[c] = 0u;
    if (const unsigned int crowded = uniform(crowded_v))
        parts += static_cast<int>(more_of(t, crowd_shift(crowded, E.n, P.n_tiles, tile_points)));
    const bool whole = parts == 1;
    if (!whole)
        for (int c = threadIdx.x; c < cells; c += kTilesBlock) weight[c] = 0u;
    uint2 sums;  // the tile's points, and the points of the event's tiles before it
    seg_pre[threadIdx.x] = block_prefix2<kTWaves>(make_uint2(len, from), scratch[0], sums).x;
    seg_from[threadIdx.x] = threadIdx.x * static_cast<unsigned int>(span) + from;
    const unsigned int n_tile = sums.x;
    if (threadIdx.x == 0) seg_pre[kBinMaxShares] = n_tile;
    const unsigned int first_row = static_cast<unsigned int>(E.row0) + sums.y;
    __syncthreads();
    const uint2 *__restrict__ mine = ents + E.row0;
    // The part's shares and points.
    auto first_share = [&](int k) {  // the first share that starts at the k-th part or later
        const unsigned int from = static_cast<unsigned int>(static_cast<unsigned long long>(n_tile) * k / parts);
        int lo = 0, hi = shares;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (seg_pre[mid] < from) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    unsigned int q_from = 0, q_to = n_tile;
    int s_from = 0;
    if (!whole) {
        s_from = first_share(part);
        const int s_to = part + 1 == parts ? shares : first_share(part + 1);
        q_from = seg_pre[s_from];
        q_to = seg_pre[s_to];
    }
    // The tile's q-th point: its row in the event, and its cell in the tile.
    auto point = [&](unsigned int q, unsigned int &cell) {
        int lo = 0, hi = shares - 1;  // the last share that starts at or before it
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (seg_pre[mid] <= q) lo = mid;
            else hi = mid - 1;
        }
        const uint2 x = mine[seg_from[lo] + (q - seg_pre[lo])];
        int u[kMaxAxes];
        unpack_cell(x.y, P.axes, u);
        cell = cell_key(u, P) - key0;
        return x;
    };
    auto fetch = [&](uint2 x, float (&row)[DP]) {
        if (vec4) {
            const float4 *src = reinterpret_cast<const float4 *>(E.pts + static_cast<size_t>(x.x) * d);
#pragma unroll
            for (int k = 0; k < DP / 4; ++k) {
                float4 w = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (4 * k < d) w = src[k];
                row[4 * k] = w.x;
                row[4 * k + 1] = w.y;
                row[4 * k + 2] = w.z;
                row[4 * k + 3] = w.w;
            }
        } else {
            const float *src = E.pts + static_cast<size_t>(x.x) * d;
#pragma unroll
            for (int k = 0; k < DP; ++k) row[k] = k < d ? src[k] : 0.0f;
        }
    };
    // A thread's first kHeld points stay in registers between the two passes, narrow
    // rows with them: they are requested here, and arrive while the cells are counted.
    constexpr int kHeld = 2;
    constexpr bool kRowsAhead = DP <= 12;
    uint2 held[kHeld];
    unsigned int held_cell[kHeld];
    float held_row[kRowsAhead ? kHeld : 1][DP];
#pragma unroll
    for (int m = 0; m < kHeld; ++m) {
        const unsigned int q = m * kTilesBlock + threadIdx.x;
        if (whole && q < n_tile) {
            held[m] = point(q, held_cell[m]);
            if (kRowsAhead) fetch(held[m], held_row[m]);
            atomicAdd(&cursor[held_cell[m]], 1u);
        }
    }
    if (whole) {
        for (unsigned int q = kHeld * kTilesBlock + threadIdx.x; q < n_tile; q += kTilesBlock) {
            unsigned int cell;
            point(q, cell);
            atomicAdd(&cursor[cell], 1u);
        }
    } else {
        // Sixteen lanes a share (a line of its entries), as many loads in flight as a share
        // of a crowded tile has use for.
        constexpr unsigned int kLanes = 16, kAhead = 8;
        const unsigned int l = threadIdx.x % kLanes;
        for (int s = threadIdx.x / kLanes; s < shares; s += kTilesBlock / kLanes) {
            const unsigned int n_seg = seg_pre[s + 1] - seg_pre[s];
            const uint2 *seg = mine + seg_from[s];
            unsigned int *to = s < s_from ? cursor : weight;
            for (unsigned int o = l; o < n_seg; o += kLanes * kAhead) {
                unsigned int pc[kAhead];
#pragma unroll
                for (unsigned int u = 0; u < kAhead; ++u)
                    if (o + kLanes * u < n_seg) pc[u] = seg[o + kLanes * u].y;
#pragma unroll
                for (unsigned int u = 0; u < kAhead; ++u) {
                    if (o + kLanes * u >= n_seg) continue;
                    int c[kMaxAxes];
                    unpack_cell(pc[u], P.axes, c);
                    atomicAdd(&to[cell_key(c, P) - key0], 1u);
                }
            }
        }
    }
    __syncthreads();
    // Points and weight before each cell: consecutive cells per thread.
    const int per = (cells + kTilesBlock - 1) / kTilesBlock;
    const int c0 = min(static_cast<int>(threadIdx.x) * per, cells), c1 = min(c0 + per, cells);
    uint2 run = make_uint2(0u, 0u);
    for (int c = c0; c < c1; ++c) {
        const unsigned int v = cursor[c] + (whole ? 0u : weight[c]);
        run.x += v;
        run.y += v + (v ? kTileWeight : 0u);
    }
    uint2 all;
    run = block_prefix2<kTWaves>(run, scratch[1], all);
    for (int c = c0; c < c1; ++c) {
        const unsigned int first = cursor[c], v = first + (whole ? 0u : weight[c]);
        cursor[c] = run.x + (whole ? 0u : first);  // past the points of earlier parts
        weight[c] = run.y;
        run.x += v;
        run.y += v + (v ? kTileWeight : 0u);
    }
    __syncthreads();
    if (part == 0) {
        for (int c = threadIdx.x; c < cells; c += kTilesBlock) cell_start[E.cell0 + key0 + c] = first_row + cursor[c];
        if (t == P.n_tiles - 1 && threadIdx.x == 0)
            cell_start[E.cell0 + P.n_cells] = static_cast<unsigned int>(E.row0) + static_cast<unsigned int>(E.n);
    }
    if (n_tile && part == 0) {
        // Pieces k with first_row <= k rows / n_pieces < first_row + n_tile.
        const unsigned long long np = static_cast<unsigned long long>(n_pieces);
        const unsigned long long R = static_cast<unsigned long long>(rows);
        const unsigned long long w_tile = all.y;
        const unsigned long long k0 = floor_div(first_row * np + R - 1, R);
        const unsigned long long k1 = floor_div((first_row + static_cast<unsigned long long>(n_tile)) * np + R - 1, R);
        for (unsigned long long k = k0 + threadIdx.x; k < k1; k += kTilesBlock) {
            // Share of the tile before the piece's ideal start, of its weight.
            const unsigned long long past_rows = floor_div(k * R, np) - first_row;
            const unsigned int at = static_cast<unsigned int>(floor_div(past_rows * w_tile, n_tile));
            int lo = 0, hi = cells - 1;  // the last cell that starts at or before it
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (weight[mid] <= at) lo = mid;
                else hi = mid - 1;
            }
            const unsigned int past = at - weight[lo];
            wave_start[k] = first_row + cursor[lo] + (past > kTileWeight ? past - kTileWeight : 0u);
        }
    }
    __syncthreads();
    // The rows, each to the next place of its cell.
    auto place = [&](uint2 x, unsigned int cell, const float (&row)[DP]) {
        const unsigned int slot = first_row + atomicAdd(&cursor[cell], 1u);
        SortedRows<DP>::store(sorted, rows, slot, row);
        reinterpret_cast<uint2 *>(sorted_id)[slot] =
            make_uint2(static_cast<unsigned int>(E.row0) + x.x, x.y);
    };
#pragma unroll
    for (int m = 0; m < kHeld; ++m)
        if (whole && m * kTilesBlock + threadIdx.x < n_tile) {
            if (!kRowsAhead) fetch(held[m], held_row[kRowsAhead ? m : 0]);
            place(held[m], held_cell[m], held_row[kRowsAhead ? m : 0]);
        }
    for (unsigned int q = (whole ? kHeld * kTilesBlock : q_from) + threadIdx.x; q < q_to; q += kTilesBlock) {
        unsigned int cell;
        const uint2 x = point(q, cell);
        float row[DP];
        fetch(x, row);
        place(x, cell, row);
    }
}

// ------------------------------------------------------------ neighbour runs

// Event of a row: the last event whose first row is <= row (empty events share
// their first row with the next event, so they are never returned for a row).
__device__ __forceinline__ int find_event(const EventDesc *__restrict__ ev, int n_events, long long row) {
    int lo = 0, hi = n_events - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (ev[mid].row0 <= row) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The neighbour cells of a cell are the cells at most R = reach cells away along
// every binned axis.  Along axis 0 (the fastest in cell order) each group of them
// is contiguous, so they form (2R+1)^(axes-1) runs of candidate rows.
__device__ __forceinline__ int run_count(const Plan &P) {
    const int side = 2 * P.reach + 1;
    return P.axes == 4 ? side * side * side : side * side;
}

// Offsets along axes 1..3 of the run a lane builds (lanes below run_count, of each half
// of the wave when the halves build the runs of two cells), and what they add to the
// key of a cell.
struct RunLane {
    int a[3];
    int key;
    bool live;
    unsigned int stride[3];  // keys between neighbours along axes 1..3 (24 bits: see wave_runs)
};

__device__ __forceinline__ RunLane run_lane(const Plan &P, bool halves) {
    const int R = P.reach, side = 2 * R + 1, t = halves ? lane_id() & 31 : lane_id();
    RunLane rl;
    rl.live = t < run_count(P);
    rl.a[0] = t % side - R;
    rl.a[1] = (t / side) % side - R;
    rl.a[2] = P.axes == 4 ? t / (side * side) - R : 0;
    rl.key = ((rl.a[2] * P.G[2] + rl.a[1]) * P.G[1] + rl.a[0]) * P.G[0];
    rl.stride[0] = static_cast<unsigned int>(P.G[0]);
    rl.stride[1] = static_cast<unsigned int>(P.G[0] * P.G[1]) & 0xffffffu;
    rl.stride[2] = static_cast<unsigned int>(P.G[0] * P.G[1] * P.G[2]) & 0xffffffu;
    return rl;
}

// Lane t < run_count builds run t around the cell whose packed coordinates are pc
// (global keys start at cell0): its first sorted row (start) and its candidates
// [pre, end) in the cell's candidate numbering (other lanes: an empty run at the end).
// With `halves`, lanes 32.. do the same for a second cell (their pc), numbered by
// itself.  Call with the whole wave active; a cell's candidate count is `end` in the
// last lane of its half (or of the wave).
// FOUR: the plan has four binned axes (and then reach 1).
template <bool FOUR>
__device__ __forceinline__ void wave_runs(unsigned int pc, unsigned int cell0, const Plan &P, const RunLane &rl,
                                          bool live, bool halves, const unsigned int *__restrict__ cell_start,
                                          unsigned int &start, unsigned int &pre, unsigned int &end) {
    const int R = FOUR ? 1 : P.reach;
    int u[kMaxAxes];
    unpack_cell(pc, FOUR ? 4 : P.axes, u);
    // Branch-free: every lane loads (a lane without a run reads the event's first
    // row of cells, a valid address) and keeps its run only if it is inside the grid
    // (the unsigned comparisons also reject negative coordinates).  An event has at most
    // 2^24 cells, so the products are full-rate 24-bit ones (a stride of 2^24 means that
    // the axis has one cell, and its coordinate is 0).
    const int y = u[1] + rl.a[0], z = u[2] + rl.a[1], w = u[3] + rl.a[2];
    const bool ok = live & (static_cast<unsigned int>(y) < static_cast<unsigned int>(P.G[1])) &
                    (static_cast<unsigned int>(z) < static_cast<unsigned int>(P.G[2])) &
                    (static_cast<unsigned int>(w) < static_cast<unsigned int>(P.G[3]));
    const int xlo = max(u[0] - R, 0), xhi = min(u[0] + R, P.G[0] - 1);
    const unsigned int crow = __umul24(u[1], rl.stride[0]) +
                              __umul24(u[2], rl.stride[1]) +
                              __umul24(u[3], rl.stride[2]);
    const unsigned int row = cell0 + (ok ? crow + static_cast<unsigned int>(rl.key) : 0u);
    const unsigned int s0 = cell_start[row + xlo];
    const unsigned int s1 = cell_start[row + xhi + 1];
    start = ok ? s0 : 0u;
    const unsigned int len = ok ? s1 - s0 : 0u;
    unsigned int x = len;
    x += dpp_move<kRowShr1>(x);
    x += dpp_move<kRowShr2>(x);
    x += dpp_move<kRowShr4>(x);
    x += dpp_move<kRowShr8>(x);
    x += dpp_move<kRowBcast15, 0xa>(x);
    if (!halves) x += dpp_move<kRowBcast31, 0xc>(x);
    end = x;
    pre = end - len;
}

// Numbers a cell's candidates: lane l of chunk b gets the sorted row of candidate
// b + l.  The runs that hold candidates are kept in order in LDS, each as (first row -
// first candidate); a run that starts inside a chunk marks its lane there with the
// chunk's own tag (so that nothing is cleared), and a ballot of the marks counts the
// runs up to each lane.  (Against marks spread by a prefix maximum over the wave and two
// cross-lane reads per chunk, with a tile's candidate rows masked where they arrive: the
// 300k-point 12-D search took 89 us, now 83.)
struct RunMap {
    unsigned int *off;   // [64] per wave: the runs with candidates
    unsigned int *mark;  // [64] per wave, cleared once before the first chunk
    unsigned int tag = 0;
    unsigned int first;   // first candidate of the lane's run, or kNone
    unsigned int before;  // runs kept in off that start before the next chunk
    static constexpr unsigned int kNone = 0x80000000u;  // candidates are fewer
    __device__ __forceinline__ void clear() {
        mark[lane_id()] = 0u;
        wave_lds_sync();
    }
    // The runs of wave_runs (of both halves): the ballot of those with candidates.
    __device__ __forceinline__ unsigned long long keep(unsigned int start, unsigned int pre, unsigned int end) {
        const unsigned long long some = __builtin_amdgcn_ballot_w64(end > pre);
        wave_lds_sync();
        if (end > pre) off[prefix_count(some)] = start - pre;
        return some;
    }
    // A new cell: the lanes that hold its runs, and the runs kept before them.
    __device__ __forceinline__ void begin(bool mine, unsigned int pre, unsigned int end, unsigned int runs_before) {
        first = mine && end > pre ? pre : kNone;
        before = runs_before;
    }
    // The row of candidate b + lane (of no meaning past the cell's last candidate).
    // Chunks are asked for in order.
    __device__ __forceinline__ unsigned int row(unsigned int b) {
        ++tag;
        if (first - b < 64u) mark[first - b] = tag;
        wave_lds_sync();
        const unsigned long long m = __builtin_amdgcn_ballot_w64(mark[lane_id()] == tag);
        // Runs that start at or before the lane's candidate: the marks up to its own.
        const unsigned long long above = m >> 1;
        const unsigned int base = before + static_cast<unsigned int>(m & 1ull) - 1u;
        const unsigned int k = prefix_count(above, base);
        before += static_cast<unsigned int>(__popcll(m));
        return off[k & 63u] + b + static_cast<unsigned int>(lane_id());
    }
};

// Waves per SIMD the search asks the register allocator for: a lane holds only a
// candidate's leading coordinates, so rows of up to 16 floats fit in 64
// registers (8 waves, some scalar registers spilled to vector lanes); wider rows,
// whose second stage holds the rest of a row, keep the compiler's choice (48 floats:
// held just below the 128 registers of 4 waves).
template <int DP>
constexpr int kSearchWaves = DP <= 16 ? 8 : (DP == 48 ? 4 : 1);

// SEL: the cap K is below kListCap, so a list that fits may still need the K
// nearest of its hits: the lists then also hold each hit's distance.
// FOUR: the call bins four axes, so that the shape of a cell's neighbourhood is known and
// takes no scalar registers.
template <int DP, bool SEL, bool FOUR>
__global__ __launch_bounds__(kBlock, kSearchWaves<DP>) void k_search(const float *__restrict__ sorted, long long rows,
                                                   const unsigned int *__restrict__ sorted_id,
                                                   const unsigned int *__restrict__ wave_start,
                                                   unsigned int *__restrict__ claims,
                                                   const EventDesc *__restrict__ ev, int n_events,
                                                   const unsigned int *__restrict__ cell_start,
                                                   const Plan *__restrict__ plans, float r2, int K,
                                                   unsigned int *__restrict__ kept,
                                                   unsigned int *__restrict__ temp,
                                                   unsigned int *__restrict__ long_slots,
                                                   unsigned int *__restrict__ extension, unsigned int ext_cap,
                                                   Counters *__restrict__ ctr,
                                                   SearchCounts *__restrict__ counts, int prio) {
    // Queries per batch: 16 when the lists also hold distances (their LDS would
    // otherwise cost occupancy), else kQTile.
    constexpr int kQT = SEL ? 16 : kQTile;
    static_assert(kQT < 64, "a batch and the start of the next fit in a wave's lanes");
    __shared__ __align__(16) unsigned int lst_all[kWaves][kQT * kListCap];
    __shared__ unsigned int lstd_all[SEL ? kWaves : 1][SEL ? kQT * kListCap : 1];  // D bits of each hit
    __shared__ unsigned int pre_all[SEL ? kWaves : 1][SEL ? kQT : 1];
    __shared__ unsigned int cnt_all[SEL ? kWaves : 1][SEL ? kQT : 1];
    __shared__ unsigned int qcnt_all[kWaves][kQT];  // hits of each query of the batch
    // Hits 16 .. 31 of the batch's queries: query << 8 | number, and the neighbour.
    constexpr bool kSpill = !SEL;
    constexpr int kSpillCap = search_spill(DP);
    static_assert(kSpillCap <= 64, "a lane per spilled hit");
    __shared__ uint2 spill_all[kSpill ? kWaves : 1][kSpill ? kSpillCap : 1];
    constexpr int kLead = search_lead(DP);
    const SortedRows<DP> pts(sorted, rows);
    // Coordinates kLead.. of the batch's queries, read by the second stage, for rows
    // wide enough that registers, not LDS, bound the waves per SIMD (32-float rows:
    // 29.1 us against 31.6 with the query rows loaded per entry; for 12-float rows the
    // LDS would cost a wave per SIMD: 106 us against 82 on the 300k-point event).
    constexpr bool kTailLds = DP >= 24 && !SEL;
    constexpr int kTail = DP - kLead;
    __shared__ float tail_all[kTailLds ? kWaves : 1][kTailLds ? kQT * kTail : 1];
    // Queued first-stage survivors: number in the batch << 32 | candidate's sorted row,
    // with the partial sum in racc.
    __shared__ unsigned long long ring_all[kWaves][kRing];
    __shared__ float racc_all[kWaves][kRing];
    __shared__ unsigned int off_all[kWaves][64];   // RunMap of each wave
    __shared__ unsigned int mark_all[kWaves][64];
    __shared__ unsigned long long tested_w[kWaves];
    __shared__ unsigned long long survived_w[kWaves];
    __shared__ unsigned int capped_w[kWaves];
    const unsigned int abort = ctr->abort;
    unsigned int *lst = lst_all[wave_id()];
    unsigned int *lstd = lstd_all[SEL ? wave_id() : 0];
    unsigned int capped = 0;
    unsigned int *tpre = pre_all[SEL ? wave_id() : 0];
    unsigned int *tcnt = cnt_all[SEL ? wave_id() : 0];
    unsigned int *qcnt = qcnt_all[wave_id()];
    uint2 *spill = spill_all[kSpill ? wave_id() : 0];
    float *qtail = tail_all[kTailLds ? wave_id() : 0];
    unsigned long long *ring = ring_all[wave_id()];
    float *racc = racc_all[wave_id()];
    RunMap map;
    map.off = off_all[wave_id()];
    map.mark = mark_all[wave_id()];
    map.clear();
    const int lane = lane_id();
    unsigned long long tested = 0;    // pairs examined (wave-uniform, as the next)
    unsigned long long survived = 0;  // pairs that reached the second stage

    // The queries, in cell order, are cut into a piece per wave, of equal work (its
    // cells' fixed costs plus its queries; a piece may start or end inside a cell,
    // so a dense cell is split instead of holding up one wave).
    // Workgroups are dealt to the 8 XCDs round-robin; the workgroups of one XCD
    // take a contiguous share of the pieces, so that they share their rows in its L2.
    // (Two pieces a wave, the second claimed from counters per XCD: 60k rows of 32, 48
    // and 64 floats 80.6, 74.3 and 88.5 us a call, 77.8, 71.3 and 86.3 with one; a
    // 120k-point 8-D event 63.0 against 58.6.)
    const unsigned int nb = gridDim.x;
    const unsigned int xcd = blockIdx.x % 8u;
    const unsigned int xb0 = xcd_first_block(xcd, nb);
    const unsigned int xnb = xcd_first_block(xcd + 1u, nb) - xb0;  // workgroups on this XCD
    const unsigned int xblk = blockIdx.x / 8u;              // this workgroup's number on its XCD
    const unsigned int x_first = kWaves * xb0;  // the XCD's first piece
    const unsigned int x_end = x_first + kWaves * xnb;
    // The wave's share and, of a single event, the plan are requested with the abort
    // flag (the shares' memory holds whatever it did when that is set).
    const unsigned int piece = x_first + xblk * kWaves + wave_id();
    unsigned int q_lo = wave_start[piece];
    unsigned int q_hi = wave_start[piece + 1u];
    Plan P = plans[0];
    asm volatile("" : "+s"(q_lo), "+s"(q_hi), "+s"(P.G[0]));
    if (abort) return;
    RunLane rl;
    bool halves = FOUR;  // a cell's runs fit half a wave: the runs of two cells are built at once
    unsigned int cell0 = 0;
    unsigned int ev_end = 0;  // first row after the current event
    const uint2 *__restrict__ sid = reinterpret_cast<const uint2 *>(sorted_id);
    // The queries are taken in batches of at most kQT, which end between cells unless a
    // single cell has more: lane l holds query win + l (its original row and packed
    // cell), and list slot l is its own.  First-stage survivors stay queued across the
    // batch's cells (a sparse cell holds a few queries), and the batch's lists are
    // written out together.
    unsigned int win = 0;             // sorted row of the batch's first query
    unsigned int head = 0, tail = 0;  // queued survivors [head, tail)
    unsigned int n_spilled = 0;       // hits kListCap .. kExtCap - 1 found in the batch (wave-uniform)
    // A pair that passes the full test joins the list of query q of the batch.  Call with
    // the whole wave active.
    auto keep = [&](bool pass, unsigned int q, unsigned int j, float D) {
        unsigned int pos = 0xffffffffu;
        if (pass) {
            pos = atomicAdd(&qcnt[q], 1u);
            if (pos < static_cast<unsigned int>(kListCap)) {
                lst[q * kListCap + pos] = j;
                if (SEL) lstd[q * kListCap + pos] = __float_as_uint(D);
            }
        }
        if (kSpill) {
            const bool over = pos - static_cast<unsigned int>(kListCap) < static_cast<unsigned int>(kExtCap - kListCap);
            const unsigned long long m = __builtin_amdgcn_ballot_w64(over);
            if (m != 0ull) {
                const unsigned int e = n_spilled + prefix_count(m);
                if (over && e < static_cast<unsigned int>(kSpillCap)) spill[e] = make_uint2(q << 8 | pos, j);
                n_spilled += static_cast<unsigned int>(__popcll(m));
            }
        }
    };
    // Second stage for ring entries [h, h + nb): lane l takes entry h + l and
    // adds terms kLead.. of the definition to the first stage's partial sum, in
    // the same order.  An entry names its query and the candidate's sorted row; the
    // remaining coordinates are loaded here (the chunk holds only the leading ones), so
    // entries outlive their chunk and cell.
    auto finish_rows = [&](unsigned int h, unsigned int nb) {
        survived += nb;
        wave_lds_sync();
        const bool act = static_cast<unsigned int>(lane) < nb;
        const unsigned int e = (h + lane) & (kRing - 1);
        const unsigned long long ent = act ? ring[e] : static_cast<unsigned long long>(win);
        const float a3 = act ? racc[e] : 0.0f;
        const unsigned int q = static_cast<unsigned int>(ent >> 32);
        const unsigned int s2 = static_cast<unsigned int>(ent);
        float cc[DP], qq[DP];
        pts.template load<kLead>(s2, cc);
        if (kTailLds) {
#pragma unroll
            for (int k = kLead; k < DP; ++k) qq[k] = qtail[q * kTail + (k - kLead)];
        } else {
            pts.template load<kLead>(win + q, qq);
        }
        unsigned int j2 = sorted_id[2u * static_cast<size_t>(s2)];
        const float D = add_terms<kLead, DP, DP, DP>(a3, cc, qq);
        // The id is requested with the rows, not (as the compiler would have it) in a
        // round trip of its own once a pair has passed.
        asm volatile("" : "+v"(j2));
        keep(act && D < r2 && s2 != win + q, q, j2, D);
        wave_lds_sync();
    };
    // Writes out the batch's nq lists, whose survivors are all finished; lane l takes
    // query l, whose original row is iq.  Kept counts for every query; lists that fit go
    // to their fixed place (kListCap slots per original row) as found, in 16-byte pieces,
    // and the placement pass orders every such list by neighbour id; lists of up to kExtCap
    // entries put the others in a block of the XCD's part of the extension; the sorted rows
    // of longer ones (and of those that find no room in the batch's spilled hits or in the
    // extension) are queued for the placement pass to collect again.  With the cap
    // binding (SEL and more than K hits), the entries of those lists are numbered through
    // a prefix over their lengths; each lane takes one entry, finds its query by binary
    // search, ranks it by its (D, j) key within its list (D >= 0, so its bits order like
    // the value; keys are distinct) and, if the rank is below K, writes it at that rank:
    // the list's first K slots then hold its K nearest.  The stores are scattered, but
    // everything about query i lands at places indexed by i, which the placement pass
    // then reads in order.
    auto flush = [&](unsigned int nq, unsigned int iq) {
        wave_lds_sync();
        const bool mine = static_cast<unsigned int>(lane) < nq;
        const unsigned int cnt = mine ? qcnt[lane] : 0u;
        const unsigned int Ku = static_cast<unsigned int>(K);
        const bool fits = mine && cnt <= static_cast<unsigned int>(kListCap) && (SEL || cnt <= Ku);
        bool ext = kSpill && mine && cnt > static_cast<unsigned int>(kListCap) &&
                   cnt <= min(static_cast<unsigned int>(kExtCap), Ku) &&
                   n_spilled <= static_cast<unsigned int>(kSpillCap);
        unsigned int block = 0u;
        if (ext) {
            block = atomicAdd(long_counter(claims, xcd, kExtCount), 1u);
            ext = block < ext_cap;
            block += xcd * ext_cap;
        }
        if (mine) {
            kept[iq] = ext ? kKeptExt | block << kKeptExtBits | cnt : min(cnt, Ku) | (fits ? 0u : kKeptLong);
            if (cnt > Ku) ++capped;
        }
        if (kSpill && n_spilled) {
            const unsigned int n = min(n_spilled, static_cast<unsigned int>(kSpillCap));
            const uint2 x = spill[min(static_cast<unsigned int>(lane), n - 1u)];
            const int q = static_cast<int>(x.x >> 8);
            const unsigned int to = static_cast<unsigned int>(__shfl(static_cast<int>(block), q));
            const bool yes = __shfl(ext ? 1 : 0, q) != 0;
            if (yes && static_cast<unsigned int>(lane) < n)
                extension[static_cast<size_t>(to) * kListCap + ((x.x & 255u) - kListCap)] = x.y;
        }
        if (mine && !ext) {
            if (!fits && cnt <= kWaveKeys)
                long_slots[wave_start[x_first] + atomicAdd(long_counter(claims, xcd, kLongCount), 1u)] = win + lane;
            if (!fits && cnt > kWaveKeys)
                long_slots[wave_start[x_end] - 1u - atomicAdd(long_counter(claims, xcd, kHugeCount), 1u)] = win + lane;
        }
        if ((fits && !(SEL && cnt > Ku)) || ext) {
            const uint4 *from = reinterpret_cast<const uint4 *>(lst + lane * kListCap);
            uint4 *to = reinterpret_cast<uint4 *>(temp + static_cast<size_t>(iq) * kListCap);
            for (unsigned int k = 0; 4u * k < min(cnt, static_cast<unsigned int>(kListCap)); ++k) to[k] = from[k];
        }
        if (SEL) {
            const unsigned int take = fits && cnt > Ku ? cnt : 0u;
            const unsigned int inc = wave_inclusive_scan(take);
            const unsigned int T = __builtin_amdgcn_readlane(inc, 63);
            if (mine) {
                tpre[lane] = inc - take;
                tcnt[lane] = take;
            }
            wave_lds_sync();
            for (unsigned int t0 = 0; t0 < T; t0 += 64) {
                const unsigned int t = t0 + lane;
                int lo = 0, hi = static_cast<int>(nq) - 1;  // last query whose list starts at or before t
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (tpre[mid] <= t) lo = mid;
                    else hi = mid - 1;
                }
                const unsigned int row = static_cast<unsigned int>(__shfl(static_cast<int>(iq), lo));
                if (t < T) {
                    const unsigned int cq = tcnt[lo];
                    const unsigned int *l = lst + lo * kListCap;
                    const unsigned int *ld = lstd + lo * kListCap;
                    const unsigned int x = t - tpre[lo];
                    const unsigned long long key = (static_cast<unsigned long long>(ld[x]) << 32) | l[x];
                    unsigned int sr = 0;  // the entry's rank by (D, j) in its list
                    for (unsigned int u = 0; u < cq; ++u)
                        sr += ((static_cast<unsigned long long>(ld[u]) << 32) | l[u]) < key ? 1u : 0u;
                    if (sr < Ku) temp[static_cast<size_t>(row) * kListCap + sr] = l[x];
                }
            }
        }
        n_spilled = 0u;
        wave_lds_sync();
    };
    float lead[kLead] = {};  // leading coordinates of the lane's query
    // The queries [q0, q1) of the batch, which share a cell, against the cell's M
    // candidates.
    auto search_cell = [&](unsigned int q0, unsigned int q1, unsigned int M) {
        // Candidates are fetched one chunk ahead so that their latency overlaps the
        // tests of the current chunk: each lane holds its candidate's leading
        // coordinates.  Idle lanes read row 0 (any row is a valid address) and are masked
        // out of every ballot, where the values are used and not here, so that nothing
        // waits for the load before the tests of the current chunk.
        float cn[kLead];
        unsigned int sn;
        auto fetch = [&](unsigned int b) {
            const unsigned int srow = map.row(b);
            sn = b + lane < M ? srow : 0u;
            const float *v = pts.lead_of(sn);
#pragma unroll
            for (int k = 0; k < kLead; ++k) cn[k] = v[k];
        };
        fetch(0u);
        for (unsigned int base = 0; base < M; base += 64) {
            float c[kLead];
#pragma unroll
            for (int k = 0; k < kLead; ++k) c[k] = cn[k];
            const unsigned int s = sn;
            // Lanes past the last candidate fail every first-stage test.
            if (base + lane >= M) c[0] = INFINITY;
            if (base + 64 < M) fetch(base + 64);
            for (unsigned int q = q0; q < q1; ++q) {
                // The query's leading coordinates, from the lane that holds them: scalar
                // loads would make every step wait for the ring's LDS writes too (one
                // counter covers both).
                float qc[kLead];
#pragma unroll
                for (int k = 0; k < kLead; ++k)
                    qc[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lead[k]), q));
                // First stage: kLead terms for all 64 candidates; pairs that are not
                // yet at r2 are queued (exact: the remaining terms only add).
                const float acc = add_terms<0, kLead, kLead, kLead>(0.0f, c, qc);
                const unsigned long long m1 = __builtin_amdgcn_ballot_w64(acc < r2);
                if (m1 == 0ull) continue;
                if (acc < r2) {
                    const unsigned int e = prefix_count(m1, tail) & (kRing - 1);
                    ring[e] = (static_cast<unsigned long long>(uniform(q)) << 32) | s;
                    racc[e] = acc;
                }
                tail += static_cast<unsigned int>(__popcll(m1));
                if (tail - head >= 64u) {
                    finish_rows(head, 64u);
                    head += 64u;
                }
            }
        }
        tested += static_cast<unsigned long long>(M) * (q1 - q0);
    };
    // The lane's query of a batch: its original row and packed cell, and the leading
    // coordinates of its row.
    // (16-float rows have no registers left to hold the latter ahead.)
    constexpr bool kLeadAhead = DP != 16;
    uint2 next = make_uint2(0u, 0u);
    float next_lead[kLead] = {};
    auto fetch_query = [&](unsigned int row) {
        if (row < q_hi) {
            next = sid[row];
            if (kLeadAhead) {
#pragma unroll
                for (int k = 0; k < kLead; ++k) next_lead[k] = pts.lead_of(row)[k];
            }
        }
    };
    fetch_query(q_lo + lane);
    for (win = q_lo; win < q_hi;) {
        if (win >= ev_end) {
            const int e = n_events == 1 ? 0 : find_event(ev, n_events, win);
            if (n_events > 1) P = plans[e];
            const EventDesc E = ev[e];
            cell0 = static_cast<unsigned int>(E.cell0);
            ev_end = static_cast<unsigned int>(E.row0) + static_cast<unsigned int>(E.n);
            halves = FOUR || run_count(P) <= 32;
            rl = run_lane(P, halves);
        }
        const unsigned int v_orig = next.x, v_pc = next.y;
#pragma unroll
        for (int k = 0; k < kLead; ++k)
            lead[k] = kLeadAhead ? next_lead[k]
                                 : pts.lead_of(min(win + lane, q_hi - 1u))[k];
        // The lanes that start a cell, and the batch's end: after its last whole cell
        // (a batch never crosses into the next event).
        const unsigned int n = min(min(64u, q_hi - win), ev_end - win);
        const unsigned int pc_before = dpp_move<kWaveShr1>(v_pc);  // with every lane active
        const unsigned long long starts = __builtin_amdgcn_ballot_w64((v_pc != pc_before) | (lane == 0)) &
                                          (n < 64u ? (1ull << n) - 1ull : ~0ull);
        unsigned int nq = n;
        if (n > static_cast<unsigned int>(kQT)) {
            const unsigned long long ends = (starts >> 1) & ((1ull << kQT) - 1ull);  // bit b: a batch of b + 1
            nq = ends ? 64u - static_cast<unsigned int>(__builtin_clzll(ends)) : static_cast<unsigned int>(kQT);
        }
        // The next batch's queries are requested before this one is worked off.
        const unsigned int after = win + nq;
        fetch_query(after + lane);
        if (prio) {
            // A SIMD issues the oldest ready wave first, so with every workgroup
            // resident from the start the waves dispatched last finish last and
            // the SIMD runs its final stretch with few waves.  Issue priority
            // falls as a wave works off its share (3 in the first quarter, 0 in
            // the last), so that waves behind are issued first and the waves of
            // a SIMD finish closer together.
            const unsigned int left = q_hi - win;
            const unsigned int share = q_hi - q_lo;
            if (4u * left > 3u * share) __builtin_amdgcn_s_setprio(3);
            else if (4u * left > 2u * share) __builtin_amdgcn_s_setprio(2);
            else if (4u * left > share) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
        if (lane < kQT) qcnt[lane] = 0u;
        if (kTailLds)
            for (unsigned int k = lane; k < nq * kTail; k += 64u)
                qtail[k] = pts.at(win + k / kTail, kLead + k % kTail);
        // End of the cell that query t of the batch lies in.
        auto cell_end = [&](unsigned int t) {
            const unsigned long long rest = t < 63u ? starts >> (t + 1u) : 0ull;
            const unsigned int e = rest ? t + 1u + static_cast<unsigned int>(__builtin_ctzll(rest)) : 64u;
            return min(e, nq);
        };
        for (unsigned int t0 = 0; t0 < nq;) {
            // The runs of this cell and, in the other half of the wave, of the next.
            const unsigned int t1 = cell_end(t0);
            const bool two = (FOUR || halves) && t1 < nq;
            const unsigned int t2 = two ? cell_end(t1) : t1;
            const unsigned int pc0 = __builtin_amdgcn_readlane(v_pc, t0);
            const unsigned int pc1 = __builtin_amdgcn_readlane(v_pc, two ? t1 : t0);
            const bool second = (FOUR || halves) && lane >= 32;
            unsigned int start, pre, end;
            wave_runs<FOUR>(second ? pc1 : pc0, cell0, P, rl, rl.live && (!second || two), FOUR || halves, cell_start, start,
                      pre, end);
            const unsigned long long some = map.keep(start, pre, end);
            const unsigned int m_first = __builtin_amdgcn_readlane(end, FOUR || halves ? 31 : 63);
            const unsigned int m_second = lane63(end);
            map.begin(!second, pre, end, 0u);
#pragma clang loop unroll(disable)
            for (unsigned int M = m_first, q = t0, qe = t1;;) {
                search_cell(q, qe, M);
                if (qe == t2) break;
                q = t1;
                qe = t2;
                M = m_second;
                map.begin(second, pre, end, static_cast<unsigned int>(__popcll(some & 0xffffffffull)));
            }
            t0 = t2;
        }
        if (tail != head) {
            finish_rows(head, tail - head);
            head = tail;
        }
        flush(nq, v_orig);
        win = after;
    }
    capped = wave_sum(capped);
    if (lane == 0) {
        tested_w[wave_id()] = tested;
        survived_w[wave_id()] = survived;
        capped_w[wave_id()] = capped;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0, sv = 0;
        unsigned int c = 0;
        for (int w = 0; w < kWaves; ++w) {
            t += tested_w[w];
            sv += survived_w[w];
            c += capped_w[w];
        }
        SearchCounts out;
        out.tested = t;
        out.survived = sv;
        out.capped = c;
        out.pad = 0u;
        counts[blockIdx.x] = out;
    }
}

// --------------------------------------------------------------- kept totals

// Kept counts summed per placement tile and per group of kKeptGroup tiles: block g
// reads group g's counts, four per lane and load and all of a lane's loads issued
// together, and writes each tile's prefix inside the group and the group's total, so
// that a row's output position is the totals of the groups before it (a few loads for
// a whole wave), its tile's prefix and the counts before it in its tile.  The workgroups
// past the groups sum the search's per-workgroup counts for the report, beside the others
// and off the placement pass's path.
__global__ __launch_bounds__(kSumsBlock) void k_kept_sums(long long n, const unsigned int *__restrict__ kept,
                                                          unsigned long long *__restrict__ tile_pre,
                                                          unsigned long long *__restrict__ group_sum, int tiles_kept,
                                                          const SearchCounts *__restrict__ counts,
                                                          int search_blocks, int groups,
                                                          Counters *__restrict__ ctr) {
    constexpr int kSumsWaves = kSumsBlock / 64;
    constexpr int kTilesPerWave = kKeptGroup / kSumsWaves;
    static_assert(kTilesPerWave * kSumsWaves == kKeptGroup && kPlaceTile == 256, "four counts per lane and tile");
    if (static_cast<int>(blockIdx.x) >= groups) {
        if (ctr->abort) return;
        __shared__ unsigned long long red[3][kSumsWaves];
        unsigned long long t = 0, sv = 0, cp = 0;
        const int step = (static_cast<int>(gridDim.x) - groups) * kSumsBlock;
        for (int k = (static_cast<int>(blockIdx.x) - groups) * kSumsBlock + static_cast<int>(threadIdx.x);
             k < search_blocks; k += step) {
            t += counts[k].tested;
            sv += counts[k].survived;
            cp += counts[k].capped;
        }
        t = wave_sum(t);
        sv = wave_sum(sv);
        cp = wave_sum(cp);
        if (lane_id() == 0) {
            red[0][wave_id()] = t;
            red[1][wave_id()] = sv;
            red[2][wave_id()] = cp;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            t = sv = cp = 0;
            for (int w = 0; w < kSumsWaves; ++w) {
                t += red[0][w];
                sv += red[1][w];
                cp += red[2][w];
            }
            // Cleared by the bounds pass; one workgroup per 2,048 counts adds to them.
            atomicAdd(&ctr->tested, t);
            atomicAdd(&ctr->survived, sv);
            if (cp) atomicAdd(&ctr->capped, static_cast<unsigned int>(cp));
        }
        return;
    }
    __shared__ unsigned int tile_sum[kKeptGroup];
    const int t0 = static_cast<int>(blockIdx.x) * kKeptGroup + wave_id() * kTilesPerWave;
    uint4 c[kTilesPerWave];
#pragma unroll
    for (int k = 0; k < kTilesPerWave; ++k) {
        const long long i = static_cast<long long>(t0 + k) * kPlaceTile + 4 * lane_id();
        if (i + 4 <= n) {
            c[k] = *reinterpret_cast<const uint4 *>(kept + i);
        } else {
            c[k].x = i < n ? kept[i] : 0u;
            c[k].y = i + 1 < n ? kept[i + 1] : 0u;
            c[k].z = i + 2 < n ? kept[i + 2] : 0u;
            c[k].w = 0u;
        }
    }
    // A tile holds at most 256 x 4096 edges and a group 64 times that: 32 bits do.
#pragma unroll
    for (int k = 0; k < kTilesPerWave; ++k) {
        const unsigned int v = kept_count(c[k].x) + kept_count(c[k].y) + kept_count(c[k].z) + kept_count(c[k].w);
        const unsigned int t = wave_sum(v);
        if (lane_id() == 0) tile_sum[wave_id() * kTilesPerWave + k] = t;
    }
    __syncthreads();
    if (wave_id() == 0) {
        const unsigned int v = tile_sum[lane_id()];
        const unsigned int inc = wave_inclusive_scan(v);
        const int t = static_cast<int>(blockIdx.x) * kKeptGroup + lane_id();
        if (t < tiles_kept) tile_pre[t] = inc - v;
        if (lane_id() == 63) group_sum[blockIdx.x] = inc;
    }
}

// --------------------------------------------------------------- long lists

// LDS of the long-list collection (besides the hit keys and the kept ids, which
// use the placement pass's window arrays: they hold nothing at that point).
template <int DP>
struct LongLds {
    unsigned int hist[256];
    __align__(16) float qv[DP];
    unsigned int run_start[64];
    unsigned int run_pre[65];
    unsigned int fill;
    unsigned int left;
    unsigned long long prefix;
};

// Sorts R values per lane ascending, element r of lane l at position 64 r + l, by a
// bitonic network: exchanges at distances of 64 and more stay inside a lane.  SIZE below
// 64 sorts each group of that many lanes by itself.  FROM = SIZE runs the last stage
// alone, which sorts values that rise and then fall.
template <int R, int SIZE = 64 * R, int FROM = 2>
__device__ __forceinline__ void wave_sort(unsigned int (&v)[R]) {
    const unsigned int lane = static_cast<unsigned int>(lane_id());
#pragma unroll
    for (unsigned int k = FROM; k <= static_cast<unsigned int>(SIZE); k <<= 1) {
#pragma unroll
        for (unsigned int j = k >> 1; j > 0; j >>= 1) {
            if (j >= 64u) {
#pragma unroll
                for (unsigned int r = 0; r < R; ++r) {
                    const unsigned int o = r ^ (j / 64u);
                    if (o > r) {
                        const unsigned int lo = min(v[r], v[o]), hi = max(v[r], v[o]);
                        const bool up = ((r * 64u) & k) == 0u;  // k >= 128 here
                        v[r] = up ? lo : hi;
                        v[o] = up ? hi : lo;
                    }
                }
            } else {
#pragma unroll
                for (unsigned int r = 0; r < R; ++r) {
                    const unsigned int p = static_cast<unsigned int>(__shfl_xor(static_cast<int>(v[r]), j));
                    const bool up = (((r * 64u) | lane) & k) == 0u || k == static_cast<unsigned int>(SIZE);
                    const bool low = (lane & j) == 0u;
                    v[r] = up == low ? min(v[r], p) : max(v[r], p);
                }
            }
        }
    }
}

// Loads h ids from LDS, sorts them and writes them local to their event.
template <int R>
__device__ __forceinline__ void wave_emit(const unsigned int *ids, unsigned int h, long long row0,
                                          long long *__restrict__ out) {
    unsigned int v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const unsigned int e = 64u * r + static_cast<unsigned int>(lane_id());
        v[r] = e < h ? ids[e] : 0xffffffffu;
    }
    wave_sort<R>(v);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const unsigned int e = 64u * r + static_cast<unsigned int>(lane_id());
        if (e < h) out[e] = static_cast<long long>(v[r]) - row0;
    }
}

// Hit keys a long list keeps in LDS (the two window arrays of the placement pass);
// a list with more hits is selected by enumerating its candidates again per pass.
constexpr unsigned int kKeyCap = kPlaceWords / 2;

// One list of more than kWaveKeys hits, collected again by the whole workgroup (every
// thread calls this with the same arguments): the query's candidates are enumerated over the same
// runs of cells as in the search and its hits keyed (bits(D) << 32 | j), which
// orders them by (D, j) since D is never negative.  With more hits than n_out
// (the cap binds) the n_out-th smallest key is found by an MSB-first radix select
// (8 passes of 8 bits; in each pass a scan over the 256 bin counts finds the bin
// that holds it), over the keys in LDS or, past kKeyCap hits, by enumerating the
// candidates again.  A list below the cap keeps all its hits, whose ids alone are
// collected.  The ids are sorted by a bitonic network whose exchanges at distances
// below 512 stay in a wave's registers (up to 512 ids by one wave), and written, local
// to the query's event, to out[0, n_out).
template <int DP>
__device__ void long_list(const SortedRows<DP> &pts, const unsigned int *__restrict__ sorted_id,
                          const unsigned int *__restrict__ cell_start, const Plan &P, unsigned int cell0,
                          unsigned int slot, float r2, unsigned int n_out, unsigned int K, long long row0,
                          long long *__restrict__ out, unsigned int *__restrict__ wbuf,
                          unsigned long long *__restrict__ scratch, LongLds<DP> &L) {
    unsigned long long *keys = reinterpret_cast<unsigned long long *>(wbuf);  // [kKeyCap]
    unsigned int *ids = wbuf;                                                  // [kMaxK], after the keys are read
    const int nruns = run_count(P);
    for (int k = threadIdx.x; k < DP; k += kPlaceBlock)
        L.qv[k] = pts.at(slot, k);
    if (wave_id() == 0) {
        unsigned int start, pre, end;
        const RunLane rl = run_lane(P, false);
        wave_runs<false>(sorted_id[2u * slot + 1u], cell0, P, rl, rl.live, false, cell_start, start, pre, end);
        const unsigned int M = lane63(end);
        L.run_start[lane_id()] = start;
        L.run_pre[lane_id()] = pre;
        if (lane_id() == 0) {
            L.run_pre[64] = M;
            L.fill = 0u;
        }
    }
    __syncthreads();
    const unsigned int M = L.run_pre[64];
    float q[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k) q[k] = L.qv[k];

    // Candidate m lies in the last run that starts at or before it (runs are
    // numbered in order, so their starts ascend).
    auto hit_key = [&](unsigned int m, bool &ok) -> unsigned long long {
        int lo = 0, hi = nruns - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (L.run_pre[mid] <= m) lo = mid;
            else hi = mid - 1;
        }
        const unsigned int s = L.run_start[lo] + (m - L.run_pre[lo]);
        float c[DP];
        pts.template load<0>(s, c);
        const float D = sq_dist<DP>(c, q);
        ok = (D < r2) && (s != slot);
        return (static_cast<unsigned long long>(__float_as_uint(D)) << 32) | sorted_id[2u * s];
    };
    // One radix pass: the bin of the left-th smallest key among those matching the
    // prefix above `shift + 8`, and how many of them lie in lower bins.
    auto pick_bin = [&](unsigned long long prefix, int shift) {
        const unsigned int c = L.hist[threadIdx.x];
        const unsigned int left = L.left;  // read before the scan's barriers; the winner writes after them
        const unsigned int below = static_cast<unsigned int>(block_exclusive_scan(c, scratch));
        if (below < left && left <= below + c) {
            L.left = left - below;
            L.prefix = prefix | (static_cast<unsigned long long>(threadIdx.x) << shift);
        }
        __syncthreads();
    };

    // Every hit into LDS, keyed (as many as fit) or, below the cap, its id alone.
    const bool all = n_out < K;
    for (unsigned int m = threadIdx.x; m < M; m += kPlaceBlock) {
        bool ok;
        const unsigned long long key = hit_key(m, ok);
        if (ok) {
            const unsigned int pos = atomicAdd(&L.fill, 1u);
            if (all) {
                if (pos < static_cast<unsigned int>(kMaxK)) ids[pos] = static_cast<unsigned int>(key);
            } else if (pos < kKeyCap) {
                keys[pos] = key;
            }
        }
    }
    __syncthreads();
    const unsigned int h = L.fill;
    const bool in_lds = h <= kKeyCap;
    unsigned long long limit = ~0ull;  // keep hits with key <= limit
    if (!all && h > n_out) {
        if (threadIdx.x == 0) {
            L.prefix = 0ull;
            L.left = n_out;
        }
        for (int pass = 0; pass < 8; ++pass) {
            const int shift = 56 - 8 * pass;
            L.hist[threadIdx.x] = 0u;
            __syncthreads();
            const unsigned long long prefix = L.prefix;
            auto count = [&](unsigned long long key) {
                if (pass == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8)))
                    atomicAdd(&L.hist[(key >> shift) & 255ull], 1u);
            };
            if (in_lds) {
                for (unsigned int k = threadIdx.x; k < h; k += kPlaceBlock) count(keys[k]);
            } else {
                for (unsigned int m = threadIdx.x; m < M; m += kPlaceBlock) {
                    bool ok;
                    const unsigned long long key = hit_key(m, ok);
                    if (ok) count(key);
                }
            }
            __syncthreads();
            pick_bin(prefix, shift);
        }
        limit = L.prefix;
    }
    // The kept ids, compacted into LDS (keys in LDS are read into registers first,
    // since the ids overwrite them).
    constexpr int kPer = kKeyCap / kPlaceBlock;
    if (all) {
        // already there
    } else if (in_lds) {
        unsigned long long mine[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const unsigned int k = threadIdx.x + static_cast<unsigned int>(j) * kPlaceBlock;
            mine[j] = k < h ? keys[k] : ~0ull;
        }
        __syncthreads();
        if (threadIdx.x == 0) L.fill = 0u;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (mine[j] != ~0ull && mine[j] <= limit) {
                const unsigned int pos = atomicAdd(&L.fill, 1u);
                if (pos < static_cast<unsigned int>(kMaxK)) ids[pos] = static_cast<unsigned int>(mine[j]);
            }
        }
    } else {
        __syncthreads();
        if (threadIdx.x == 0) L.fill = 0u;
        __syncthreads();
        for (unsigned int m = threadIdx.x; m < M; m += kPlaceBlock) {
            bool ok;
            const unsigned long long key = hit_key(m, ok);
            if (ok && key <= limit) {
                const unsigned int pos = atomicAdd(&L.fill, 1u);
                if (pos < static_cast<unsigned int>(kMaxK)) ids[pos] = static_cast<unsigned int>(key);
            }
        }
    }
    __syncthreads();
    // Bitonic sort of the ids by value; slots past the ids found hold the largest
    // value (only a corrupted kept count could leave any of them in [0, n_out)).
    const unsigned int found = min(L.fill, static_cast<unsigned int>(kMaxK));
    constexpr unsigned int kChunk = 512;
    static_assert(kMaxK % kChunk == 0, "whole chunks");
    unsigned int size = kChunk;
    while (size < n_out) size <<= 1;
    for (unsigned int e = found + threadIdx.x; e < size; e += kPlaceBlock) ids[e] = 0xffffffffu;
    __syncthreads();
    if (n_out <= kChunk) {
        if (wave_id() == 0) {
            if (n_out <= 64u) wave_emit<1>(ids, n_out, row0, out);
            else if (n_out <= 128u) wave_emit<2>(ids, n_out, row0, out);
            else if (n_out <= 256u) wave_emit<4>(ids, n_out, row0, out);
            else wave_emit<kChunk / 64>(ids, n_out, row0, out);
        }
        __syncthreads();
        return;
    }
    for (unsigned int k = kChunk; k <= size; k <<= 1) {
        for (unsigned int j = k >> 1; j >= kChunk; j >>= 1) {
            for (unsigned int p = threadIdx.x; p < size / 2; p += kPlaceBlock) {
                const unsigned int e = 2u * (p & ~(j - 1u)) | (p & (j - 1u));  // the pair's lower place
                const unsigned int a = ids[e], b = ids[e + j];
                const bool up = (e & k) == 0;
                ids[e] = up ? min(a, b) : max(a, b);
                ids[e + j] = up ? max(a, b) : min(a, b);
            }
            __syncthreads();
        }
        // The rest of the stage, a chunk per wave; falling chunks as their complements.
        for (unsigned int e0 = wave_id() * kChunk; e0 < size; e0 += kWaves * kChunk) {
            const unsigned int flip = (e0 & k) == 0 ? 0u : 0xffffffffu;
            unsigned int v[kChunk / 64];
#pragma unroll
            for (int r = 0; r < static_cast<int>(kChunk / 64); ++r) v[r] = ids[e0 + 64u * r + lane_id()] ^ flip;
            if (k == kChunk) wave_sort<kChunk / 64>(v);
            else wave_sort<kChunk / 64, kChunk, kChunk>(v);
#pragma unroll
            for (int r = 0; r < static_cast<int>(kChunk / 64); ++r) ids[e0 + 64u * r + lane_id()] = v[r] ^ flip;
        }
        __syncthreads();
    }
    for (unsigned int t = threadIdx.x; t < n_out; t += kPlaceBlock) out[t] = static_cast<long long>(ids[t]) - row0;
    __syncthreads();
}

// The lists a single wave collects: at most kWaveKeys hits.

// Keeps the `want` smallest of h hits by (D, id), want < h, and compacts their ids to
// the front of ids.  The want-th smallest D is found bit by bit from the top (D >= 0,
// so its bits order like the value), counting with ballots; a step that leaves exactly
// `want` hits below ends the search, and only hits tied at that D are then told apart
// by id, in the same way.
template <int R>
__device__ __forceinline__ void wave_select(const unsigned int *dist, unsigned int *ids, unsigned int h,
                                            unsigned int want) {
    unsigned int d[R], v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const unsigned int e = 64u * r + static_cast<unsigned int>(lane_id());
        d[r] = e < h ? dist[e] : 0xffffffffu;
        v[r] = e < h ? ids[e] : 0xffffffffu;
    }
    unsigned int T = 0u;  // the largest value with fewer than `want` D bits below it
    bool split = false;
    for (int b = 30; b >= 0; --b) {
        const unsigned int c = T | (1u << b);
        unsigned int n = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) n += __popcll(__builtin_amdgcn_ballot_w64(d[r] < c));
        if (n == want) {
            T = c;
            split = true;
            break;
        }
        if (n < want) T = c;
    }
    unsigned int U = 0u;  // ties at T are kept below this id
    if (!split) {
        unsigned int below = 0, at = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            below += __popcll(__builtin_amdgcn_ballot_w64(d[r] < T));
            at += __popcll(__builtin_amdgcn_ballot_w64(d[r] == T));
        }
        const unsigned int need = want - below;
        U = 0xffffffffu;
        if (at > need) {
            U = 0u;
            for (int b = 30; b >= 0; --b) {  // ids are below 2^31
                const unsigned int c = U | (1u << b);
                unsigned int n = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) n += __popcll(__builtin_amdgcn_ballot_w64(d[r] == T && v[r] < c));
                if (n < need) U = c;
            }
            ++U;  // U was the need-th smallest id
        }
    }
    wave_lds_sync();
    unsigned int at = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool keep = d[r] < T || (d[r] == T && v[r] < U);
        const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
        if (keep) ids[at + prefix_count(m)] = v[r];
        at += static_cast<unsigned int>(__popcll(m));
    }
    wave_lds_sync();
}

// One long list, collected again by one wave: the query's candidates are enumerated
// over the same runs of cells as in the search, 64 at a time, one per lane with its
// whole row; hits go to LDS (dist and ids, kWaveKeys entries each).  With more hits
// than n_out (the cap binds) the n_out nearest are selected; the kept ids are sorted in
// registers and written, local to the query's event, to out[0, n_out).  A list takes a
// wave a few hundred instructions and no barrier, and as many lists are in flight as
// waves.  Collecting each with a whole workgroup, as the larger lists are (long_list,
// a bitonic network with a barrier per step), the placement pass took 690 us for 51,000
// lists of about 45 entries, against 53 us; 53 us against 14 on a 120k-point event
// with 3,200 lists of 17 and more, and 380 us against 31 with the nearest 32 of
// about 95 kept for 17,000 queries.  What bounds a list is its chain of round trips
// (queue, ids, counts and cells, candidates), so the LDS of the pass is kept to what
// leaves six workgroups per CU: lists of up to 512 hits and windows of 3,072 positions
// against 1,024 and 4,096 (four workgroups) took the placement of a batch of 5.6M
// points with 148,000 long lists from 560 to 458 us.
template <int DP>
__device__ __forceinline__ void wave_list(const SortedRows<DP> &pts, const unsigned int *__restrict__ sorted_id,
                          const unsigned int *__restrict__ cell_start, const Plan &P, unsigned int cell0,
                          unsigned int slot, unsigned int pc, float r2, unsigned int n_out, long long row0,
                          long long *__restrict__ out, unsigned int *dist, unsigned int *ids, RunMap &map) {
    const int lane = lane_id();
    unsigned int start, pre, end;
    const RunLane rl = run_lane(P, false);
    wave_runs<false>(pc, cell0, P, rl, rl.live, false, cell_start, start, pre, end);
    const unsigned int M = lane63(end);
    float qrow[DP];  // wave-uniform
    pts.template load<0>(slot, qrow);
    unsigned int h = 0;
    map.keep(start, pre, end);
    map.begin(true, pre, end, 0u);
    for (unsigned int b = 0; b < M; b += 64u) {
        const unsigned int mm = b + lane;
        const unsigned int srow = map.row(b);
        const unsigned int s = mm < M ? srow : slot;
        const unsigned int j = sorted_id[2u * static_cast<size_t>(s)];
        float c[DP];
        pts.template load<0>(s, c);
        const float D = sq_dist<DP>(c, qrow);
        const bool hit = D < r2 && s != slot;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(hit);
        const unsigned int pos = h + prefix_count(m);
        if (hit && pos < kWaveKeys) {  // the search counted no more hits than fit
            dist[pos] = __float_as_uint(D);
            ids[pos] = j;
        }
        h += static_cast<unsigned int>(__popcll(m));
    }
    wave_lds_sync();
    h = min(h, kWaveKeys);
    if (h > n_out) {
        if (h <= 64u) wave_select<1>(dist, ids, h, n_out);
        else if (h <= 128u) wave_select<2>(dist, ids, h, n_out);
        else if (h <= 256u) wave_select<4>(dist, ids, h, n_out);
        else wave_select<kWaveKeys / 64>(dist, ids, h, n_out);
        h = n_out;
    }
    if (h <= 64u) wave_emit<1>(ids, h, row0, out);
    else if (h <= 128u) wave_emit<2>(ids, h, row0, out);
    else if (h <= 256u) wave_emit<4>(ids, h, row0, out);
    else wave_emit<kWaveKeys / 64>(ids, h, row0, out);
    wave_lds_sync();
}

// ------------------------------------------------------------------- place

// Block b < tiles_kept owns queries [kPlaceTile b, kPlaceTile (b + 1)), one per
// thread.  Its first output position is the sum of the totals of the groups of
// kKeptGroup tiles before its own and its prefix inside its group; a block
// scan of its kept counts gives each query's offset.  Lists in the fixed
// kListCap-slot places come from the search in the order their hits were found:
// each query's thread sorts its list in registers.  The block's output is then
// formed in LDS a window at a time (each query's thread puts its row and its
// neighbours at its own positions), so that consecutive threads write consecutive
// int64 positions; the neighbour positions of a long list are left to its
// collector.  Indices are made local to each query's event.  Block 0 writes the
// report and the status; the block holding an event's first row writes its edge
// offset.  Then every block, including those past the tiles (the grid has at least
// kPlaceMinBlocks), collects the long lists of the search's queue in turn, one per
// wave, then the larger ones, one per workgroup: the list's output position is the
// totals of the groups before its query's tile, the tile's prefix in its group and the
// kept counts before the query in its tile.
template <int DP>
__global__ __launch_bounds__(kPlaceBlock) void k_place(long long rows, const EventDesc *__restrict__ ev,
                                                       int n_events, const unsigned int *__restrict__ kept,
                                                       const unsigned long long *__restrict__ tile_pre,
                                                       const unsigned long long *__restrict__ group_sum,
                                                       int groups_kept, int tiles_kept,
                                                       const unsigned int *__restrict__ long_slots,
                                                       const unsigned int *__restrict__ long_counts,
                                                       const unsigned int *__restrict__ wave_start,
                                                       unsigned int search_blocks,
                                                       const unsigned int *__restrict__ extension,
                                                       unsigned int ext_cap,
                                                       const unsigned int *__restrict__ temp,
                                                       const float *__restrict__ sorted,
                                                       const unsigned int *__restrict__ sorted_id,
                                                       const unsigned int *__restrict__ cell_start, float r2, int K,
                                                       long long *__restrict__ src, long long *__restrict__ dst,
                                                       unsigned long long cap, const Plan *__restrict__ plans,
                                                       const Counters *__restrict__ ctr,
                                                       long long *__restrict__ edge_off,
                                                       Report *__restrict__ report) {
    static_assert(kPlaceBlock == kPlaceTile, "one query per thread");
    static_assert(kPlaceWords >= kMaxK && kPlaceBlock == 256, "a long list's ids fit");
    static_assert(kPlaceWords >= 2 * static_cast<int>(kWaveKeys) * kWaves, "each wave has room for its hits");
    static_assert(4 * kPlaceWords >= 5 * kOwnerWindow, "a window takes five bytes per position");
    // A window of the block's output (neighbours, then queries as one byte each); a
    // neighbour entry of kSkip belongs to a long list, written by its collector.
    constexpr unsigned int kSkip = 0xffffffffu;
    __shared__ unsigned int o[kPlaceTile + 1];
    __shared__ __align__(16) unsigned int wbuf[kPlaceWords];
    unsigned int *wdst = wbuf;
    unsigned char *wq = reinterpret_cast<unsigned char *>(wbuf + kOwnerWindow);  // the query, in the block
    __shared__ unsigned int il_s[kPlaceTile];  // event-local row of each of the block's queries
    __shared__ uint2 ext_s[kPlaceTile];  // the block's queries with extended lists, and their kept words
    __shared__ unsigned int n_ext;
    if (threadIdx.x == 0) n_ext = 0u;    // counted after the next barrier
    __shared__ unsigned long long scratch[kWaves];
    __shared__ LongLds<DP> L;
    __shared__ unsigned int map_all[kWaves][128];  // RunMap of each wave
    __shared__ unsigned int q_first[8], q_last[8], q_wave[9], q_huge[9];
    const SortedRows<DP> pts(sorted, rows);
    const bool abort = ctr->abort != 0;
    const int b = static_cast<int>(blockIdx.x);
    const bool tile_block = b < tiles_kept;
    const long long i0 = static_cast<long long>(b) * kPlaceTile;
    const int cnt = tile_block ? static_cast<int>(rows - i0 < kPlaceTile ? rows - i0 : kPlaceTile) : 0;
    const int q = threadIdx.x;
    // The query's kept count and its list of up to kListCap (at the query's own
    // fixed place) are requested first, so that their round trips overlap the sums
    // of the tile totals below.
    // (Neither waits for the abort flag, nor the list for the count: a place that holds no
    // list is read for nothing.)
    unsigned int kraw = 0u;
    unsigned int v[kListCap];
    if (q < cnt) {
        kraw = kept[i0 + q];
        const uint4 *l4 = reinterpret_cast<const uint4 *>(temp + static_cast<size_t>(i0 + q) * kListCap);
#pragma unroll
        for (int c = 0; c < kListCap / 4; ++c) {
            const uint4 w = l4[c];
            v[4 * c] = w.x;
            v[4 * c + 1] = w.y;
            v[4 * c + 2] = w.z;
            v[4 * c + 3] = w.w;
        }
    }
    const bool mine = !abort && q < cnt;
    kraw = mine ? kraw : 0u;
    const unsigned int kq = kept_count(kraw);
    const bool is_ext = mine && (kraw & kKeptExt) != 0u;
    const bool is_long = mine && (kraw & kKeptLong) != 0u;
    const bool fixed = mine && kq > 0u && !is_long && !is_ext;
    // Kept neighbours before tile t (and all of them), one part per thread.
    auto tile_prefix = [&](int t, unsigned long long &before, unsigned long long &all) {
        const int gt = t / kKeptGroup;
        before = threadIdx.x == 0 ? tile_pre[t] : 0ull;
        all = 0;
        for (int x = threadIdx.x; x < groups_kept; x += kPlaceBlock) {
            const unsigned long long y = group_sum[x];
            all += y;
            if (x < gt) before += y;
        }
    };
    __shared__ unsigned long long red[3 * kWaves];
    unsigned long long pre = 0, tot = 0;
    if (!abort) tile_prefix(tile_block ? b : 0, pre, tot);
    // The block's first output position, E, and each query's offset in the block.
    unsigned long long oq64;
    block_sums_and_scan(pre, tot, static_cast<unsigned long long>(kq), red, pre, tot, oq64);
    const long long E = static_cast<long long>(tot);
    const bool overflow = static_cast<unsigned long long>(E) > cap;
    if (b == 0 && threadIdx.x == 0) {
        const Plan P = plans[0];
        Report rep;
        rep.n_edges = E;
        rep.tested = abort ? 0ull : ctr->tested;
        rep.survived = abort ? 0ull : ctr->survived;
        rep.abort = abort ? 1 : 0;
        rep.capped = abort ? 0u : ctr->capped;
        rep.heavy = 0u;
        for (unsigned int x = 0; x < 8u && !abort; ++x)
            rep.heavy += long_counts[x * kClaimStride + kLongCount] +
                         long_counts[x * kClaimStride + kHugeCount] +
                         min(long_counts[x * kClaimStride + kExtCount], ext_cap);
        rep.n_cells = P.n_cells;
        for (int p = 0; p < kMaxAxes; ++p) {
            rep.G[p] = P.G[p];
            rep.c[p] = P.c[p];
        }
        *report = rep;
        edge_off[n_events] = E;
        edge_off[n_events + 1] = abort ? 2 : (overflow ? 3 : 0);
    }
    if (tile_block) {
        const unsigned int oq = static_cast<unsigned int>(oq64);
        if (q < cnt) o[q] = oq;
        if (q == cnt - 1) o[cnt] = oq + kq;
        if (is_ext) ext_s[atomicAdd(&n_ext, 1u)] = make_uint2(static_cast<unsigned int>(q), kraw);
        __syncthreads();
        // Edge ranges of the events whose first row lies in this block (events with no
        // rows at the very end start at E).
        {
            int lo = 0, hi = n_events;  // first event whose first row is >= i0
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (ev[mid].row0 < i0) lo = mid + 1;
                else hi = mid;
            }
            const bool last_tile = b == tiles_kept - 1;
            for (int e = lo + threadIdx.x; e < n_events; e += kPlaceBlock) {
                const long long r0 = ev[e].row0;
                if (r0 >= i0 + cnt && !(last_tile && r0 >= rows)) break;
                edge_off[e] = abort ? 0 : (r0 >= rows ? E : static_cast<long long>(pre + o[r0 - i0]));
            }
        }
        if (abort || overflow) return;
        const unsigned int brow =
            n_events == 1 || q >= cnt ? 0u : static_cast<unsigned int>(ev[find_event(ev, n_events, i0 + q)].row0);
        const unsigned int total = o[cnt];
        if (pre + total > cap) return;  // cannot happen when E <= cap; never write past the outputs
        // A list from a fixed place holds the query's hits in the order they were
        // found: its thread sorts it (a bitonic network over 16 slots, the unused
        // ones holding the largest value).
        if (fixed) {
#pragma unroll
            for (int u = 0; u < kListCap; ++u) v[u] = static_cast<unsigned int>(u) < kq ? v[u] : 0xffffffffu;
#pragma unroll
            for (int k = 2; k <= kListCap; k <<= 1) {
#pragma unroll
                for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
                    for (int u = 0; u < kListCap; ++u) {
                        const int l = u ^ j;
                        if (l > u) {
                            const unsigned int lo = v[u] < v[l] ? v[u] : v[l];
                            const unsigned int hi = v[u] < v[l] ? v[l] : v[u];
                            const bool up = (u & k) == 0;
                            v[u] = up ? lo : hi;
                            v[l] = up ? hi : lo;
                        }
                    }
                }
            }
        }
        il_s[q] = static_cast<unsigned int>(i0 + q) - brow;
        for (unsigned int w0 = 0; w0 < total; w0 += kOwnerWindow) {
            const unsigned int wend = total - w0 < kOwnerWindow ? total - w0 : kOwnerWindow;
            if (fixed) {
#pragma unroll
                for (int u = 0; u < kListCap; ++u) {
                    const unsigned int pw = oq + static_cast<unsigned int>(u) - w0;  // wraps when before the window
                    if (static_cast<unsigned int>(u) < kq && oq + u >= w0 && pw < wend) {
                        wq[pw] = static_cast<unsigned char>(q);
                        wdst[pw] = v[u] - brow;
                    }
                }
            }
            // Positions of lists written elsewhere: up to kOwnSpan by the list's thread, more
            // by its wave.  (All by the thread alone, a call with 8,000 lists of 4,000
            // took 29.1 ms, 2.2 so; 20,000 lists of 500 1.04 and 0.51.)
            constexpr unsigned int kOwnSpan = 128;
            const bool other = is_long || is_ext;
            const unsigned int a0 = other && oq > w0 ? oq - w0 : 0u;
            const unsigned int a1 = other && oq + kq > w0 ? min(oq + kq - w0, wend) : 0u;
            const bool wide = a1 > a0 && a1 - a0 > kOwnSpan;
            if (!wide) {
                for (unsigned int pw = a0; pw < a1; ++pw) {
                    wq[pw] = static_cast<unsigned char>(q);
                    wdst[pw] = kSkip;
                }
            }
            for (unsigned long long m = __builtin_amdgcn_ballot_w64(wide); m != 0ull; m &= m - 1ull) {
                const int owner = __builtin_ctzll(m);
                const unsigned int lo = __builtin_amdgcn_readlane(a0, owner);
                const unsigned int hi = __builtin_amdgcn_readlane(a1, owner);
                for (unsigned int pw = lo + lane_id(); pw < hi; pw += 64u) {
                    wq[pw] = static_cast<unsigned char>(wave_id() * 64 + owner);
                    wdst[pw] = kSkip;
                }
            }
            __syncthreads();
            for (unsigned int pw = threadIdx.x; pw < wend; pw += kPlaceBlock) {
                const long long at = static_cast<long long>(pre) + w0 + pw;
                src[at] = il_s[wq[pw]];
                const unsigned int dv = wdst[pw];
                if (dv != kSkip) dst[at] = dv;
            }
            __syncthreads();
        }
        // Extended lists, one per half wave: the first kListCap neighbours from the query's
        // fixed place, the others from its block of the extension, sorted across 32 lanes.
        for (unsigned int x0 = 2u * wave_id(); x0 < n_ext; x0 += 2u * kWaves) {
            const unsigned int l = threadIdx.x & 31u, x = x0 + (static_cast<unsigned int>(lane_id()) >> 5);
            const uint2 w = ext_s[min(x, n_ext - 1u)];
            const unsigned int count = x < n_ext ? w.y & kKeptExtCount : 0u;
            const unsigned int block = (w.y & ~kKeptExt) >> kKeptExtBits;
            const unsigned int *from = l < static_cast<unsigned int>(kListCap)
                                           ? temp + static_cast<size_t>(i0 + w.x) * kListCap + l
                                           : extension + static_cast<size_t>(block) * kListCap + (l - kListCap);
            unsigned int id[1] = {0xffffffffu};
            if (l < count) id[0] = *from;
            wave_sort<1, 32>(id);
            const unsigned int base = static_cast<unsigned int>(i0) + w.x - il_s[w.x];  // the event's first row
            if (l < count) dst[static_cast<long long>(pre + o[w.x]) + l] = id[0] - base;
        }
    }
    if (abort || overflow) return;
    // The search's queues, one per XCD: where each starts and ends in long_slots, and
    // the lists of each kind before it.
    if (threadIdx.x < 64) {
        const unsigned int x = min(threadIdx.x, 7u);
        const unsigned int *c = long_counts + x * kClaimStride;
        const unsigned int n_wave = threadIdx.x < 8 ? c[kLongCount] : 0u;
        const unsigned int n_huge = threadIdx.x < 8 ? c[kHugeCount] : 0u;
        const unsigned int first = wave_start[kWaves * xcd_first_block(x, search_blocks)];
        const unsigned int last = wave_start[kWaves * xcd_first_block(x + 1u, search_blocks)];
        const unsigned int wave_inc = wave_scan_add(n_wave), huge_inc = wave_scan_add(n_huge);
        if (threadIdx.x < 8) {
            q_first[x] = first;
            q_last[x] = last;
            q_wave[x + 1] = wave_inc;
            q_huge[x + 1] = huge_inc;
            if (x == 0) q_wave[0] = q_huge[0] = 0u;
        }
    }
    __syncthreads();
    // Long lists that a wave collects.  A queue is about in the search's order, so
    // neighbouring entries share candidates: each XCD takes a contiguous share of them
    // all, its waves in turn.
    {
        const unsigned int xcd = blockIdx.x % 8u;
        const unsigned int xnb = gridDim.x / 8u + (xcd < gridDim.x % 8u ? 1u : 0u);
        const unsigned long long n_long = q_wave[8];
        const unsigned int lo = static_cast<unsigned int>(n_long * xcd / 8u);
        const unsigned int hi = static_cast<unsigned int>(n_long * (xcd + 1u) / 8u);
        unsigned int queue = 0;
        unsigned int *lds = wbuf + wave_id() * (2 * kWaveKeys);
        RunMap map;
        map.off = map_all[wave_id()];
        map.mark = map.off + 64;
        map.clear();
        // An entry's row, and then the row's ids, are requested while the entries before
        // it are worked off.
        const unsigned int step = xnb * kWaves;
        auto entry = [&](unsigned int h) -> unsigned int {
            if (h >= hi) return 0u;
            while (h >= q_wave[queue + 1u]) ++queue;
            const unsigned int slot = long_slots[q_first[queue] + (h - q_wave[queue])];
            return static_cast<long long>(slot) < rows ? slot : 0u;  // only a corrupted queue holds another
        };
        const uint2 *sid = reinterpret_cast<const uint2 *>(sorted_id);
        unsigned int h = lo + blockIdx.x / 8u * kWaves + wave_id();
        unsigned int slot1 = entry(h);
        unsigned int slot2 = entry(h + step);
        uint2 id1 = sid[slot1];
        long long ev_lo = 0, ev_end = 0;  // rows of the event that P and cell0 are of
        Plan P;
        unsigned int cell0 = 0;
        for (; h < hi; h += step) {
            const unsigned int slot = uniform(slot1);
            const uint2 id = id1;
            slot1 = slot2;
            slot2 = entry(h + 2u * step);
            id1 = sid[slot1];
            const long long gi = uniform(id.x);  // the query's original row
            const int t = static_cast<int>(gi / kPlaceTile);
            if (gi >= rows || t >= tiles_kept) continue;  // likewise
            // Output position: one 16-byte load per lane covers the tile's counts.
            unsigned long long at = lane_id() == 0 ? tile_pre[t] : 0ull;
            for (int x = lane_id(); x < t / kKeptGroup; x += 64) at += group_sum[x];
            const long long x0 = static_cast<long long>(t) * kPlaceTile + 4 * lane_id();
            if (x0 < gi) {  // then x0 .. x0 + 3 lie in the array (256-byte aligned, padded)
                const uint4 c = *reinterpret_cast<const uint4 *>(kept + x0);
                at += kept_count(c.x);
                if (x0 + 1 < gi) at += kept_count(c.y);
                if (x0 + 2 < gi) at += kept_count(c.z);
                if (x0 + 3 < gi) at += kept_count(c.w);
            }
            const unsigned int nq = kept_count(uniform(kept[gi]));
            if (gi < ev_lo || gi >= ev_end) {
                const int e = n_events == 1 ? 0 : find_event(ev, n_events, gi);
                P = plans[e];
                cell0 = static_cast<unsigned int>(ev[e].cell0);
                ev_lo = ev[e].row0;
                ev_end = ev_lo + ev[e].n;
            }
            at = wave_sum(at);
            if (at + nq > cap) continue;  // cannot happen when E <= cap
            wave_list<DP>(pts, sorted_id, cell_start, P, cell0, slot, uniform(id.y), r2, nq, ev_lo, dst + at, lds,
                          lds + kWaveKeys, map);
        }
    }
    __syncthreads();
    // Larger ones, collected by the whole workgroup, every gridDim-th one.
    const unsigned int n_huge = q_huge[8];
    unsigned int huge_queue = 0;
    for (unsigned int h = blockIdx.x; h < n_huge; h += gridDim.x) {
        while (h >= q_huge[huge_queue + 1u]) ++huge_queue;
        const unsigned int slot = long_slots[q_last[huge_queue] - 1u - (h - q_huge[huge_queue])];
        if (static_cast<long long>(slot) >= rows) continue;  // only a corrupted queue
        const long long gi = sorted_id[2u * slot];  // the query's original row
        const int t = static_cast<int>(gi / kPlaceTile);
        if (gi >= rows || t >= tiles_kept) continue;  // likewise
        unsigned long long at = 0, all = 0;
        tile_prefix(t, at, all);
        const long long x = static_cast<long long>(t) * kPlaceTile + threadIdx.x;
        if (x < gi) at += kept_count(kept[x]);
        at = block_sum(at, scratch);
        const unsigned int nq = kept_count(kept[gi]);
        if (at + nq > cap) continue;  // cannot happen when E <= cap
        const int e = n_events == 1 ? 0 : find_event(ev, n_events, gi);
        const Plan P = plans[e];
        long_list<DP>(pts, sorted_id, cell_start, P, static_cast<unsigned int>(ev[e].cell0), slot, r2, nq,
                      static_cast<unsigned int>(K), ev[e].row0, dst + at, wbuf, scratch, L);
    }
}

// The binning through tiles works in memory of the other one: the entries where packed
// cells and ranks lie (next to each other), the tables in the histogram.
uint2 *bin_ents(const Workspace &ws) { return reinterpret_cast<uint2 *>(ws.pcell); }
unsigned short *bin_table(const Workspace &ws) { return reinterpret_cast<unsigned short *>(ws.cell_count); }
unsigned int *crowd_counts(const Workspace &ws) { return ws.kept; }
unsigned long long *crowd_sums(const Workspace &ws) { return reinterpret_cast<unsigned long long *>(ws.edge_off); }

// Binning through tiles in a one-dimensional grid (event_block): where the largest event
// has more than kFlatFrom times the mean.  Whole synchronous batches, two and one
// dimensions: 200k points with 300 events of 50 502 and 315 us (29 times the mean), 300k
// with 20 of 20k 278 and 262 (9), 100k with 10 of 10k 148 and 141 (5.5), 200k with 3 of
// 100k 221 and 211 (1.6), 64 events of 20k to 150k 1,370 both ways.
constexpr long long kFlatFrom = 2;
bool flat_grid(const LaunchArgs &a, long long rows) {
    return a.n_events > 1 && static_cast<long long>(a.max_n) * a.n_events > kFlatFrom * rows;
}

// Launches the stages whose kernels depend on the padded row width.
template <int DP>
void launch_rows(const LaunchArgs &a, const Workspace &ws, int vec4) {
    auto mark = [&](int stage) {
        if (a.events) (void)hipEventRecord(a.events[stage], a.stream);
    };
    const long long rows = ws.rows;
    const long long nb = (static_cast<long long>(a.max_n) + kBlock - 1) / kBlock;
    const int gs = static_cast<int>(nb < 1 ? 1 : (nb > 4096 ? 4096 : nb));
    if (a.bin_span) {
        // An odd number of blocks an event: they are dealt to the XCDs in turn, so that with a
        // multiple of 8 the events' first tiles, in small events the only ones with points,
        // would all go to one XCD (2,000 events of one point: 31 us with 9 blocks each, 43
        // with 10, 87 with 8).
        const int flat = flat_grid(a, rows) ? a.n_events : 0;
        const dim3 grid = flat ? dim3(static_cast<unsigned int>(
                                     blocks_before(rows, a.n_events, tile_block_rows(a.tile_points), kTilesExtra) + 1))
                               : dim3(tile_blocks(a.max_n, a.tile_points) | 1, a.n_events);
        hipLaunchKernelGGL(k_tiles<DP>, grid, dim3(kTilesBlock), 0, a.stream, a.d, vec4, a.bin_span, ws.ev, a.ev0,
                           a.ev_from_arg, flat, a.tile_points, ws.plans,
                           bin_ents(ws), bin_table(ws), crowd_counts(ws),
                           a.max_n < crowd_least(a.tile_points) ? nullptr : crowd_sums(ws), ws.cell_start, ws.sorted,
                           ws.sorted_id, ws.wave_start,
                           a.search_blocks * kWaves, ws.rows, ws.claims);
    } else {
        hipLaunchKernelGGL(k_scatter<DP>, dim3(gs, a.n_events), dim3(kBlock), 0, a.stream, a.d, vec4, ws.ev, a.ev0,
                           a.ev_from_arg, ws.plans,
                           ws.pcell, ws.rank, ws.cell_start, ws.ctr, ws.sorted, rows, ws.sorted_id);
    }
    mark(4);
    // The extension's blocks take the memory of the histogram (or of the binning's tables),
    // read for the last time before the search: an eighth each XCD.
    const unsigned int ext_cap =
        static_cast<unsigned int>(std::min<long long>(ws.cells / kListCap, kExtBlocksMax) / 8);
    SearchCounts *counts = reinterpret_cast<SearchCounts *>(ws.rank);
    auto search = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(a.search_blocks), dim3(kBlock), 0, a.stream, ws.sorted, rows, ws.sorted_id,
                           ws.wave_start, ws.claims, ws.ev, a.n_events, ws.cell_start, ws.plans, a.r2, a.K, ws.kept,
                           ws.temp, ws.long_slots, ws.cell_count, ext_cap, ws.ctr, counts, a.search_prio);
    };
    if (a.K < kListCap) a.axes == 4 ? search(k_search<DP, true, true>) : search(k_search<DP, true, false>);
    else a.axes == 4 ? search(k_search<DP, false, true>) : search(k_search<DP, false, false>);
    mark(5);
    // One block per group of tiles, and one per 2,048 counts of the search.
    hipLaunchKernelGGL(k_kept_sums, dim3(ws.groups_kept_n + (a.search_blocks + 2047) / 2048), dim3(kSumsBlock), 0,
                       a.stream, rows, ws.kept, ws.sums_kept, ws.sums_kept2, ws.tiles_kept_n, counts,
                       a.search_blocks, ws.groups_kept_n, ws.ctr);
    mark(6);
    const int place_blocks = ws.tiles_kept_n > kPlaceMinBlocks ? ws.tiles_kept_n : kPlaceMinBlocks;
    hipLaunchKernelGGL(k_place<DP>, dim3(static_cast<unsigned int>(place_blocks)), dim3(kPlaceBlock), 0, a.stream,
                       rows, ws.ev, a.n_events, ws.kept, ws.sums_kept, ws.sums_kept2, ws.groups_kept_n,
                       ws.tiles_kept_n, ws.long_slots, ws.claims, ws.wave_start,
                       static_cast<unsigned int>(a.search_blocks), ws.cell_count, ext_cap, ws.temp, ws.sorted, ws.sorted_id, ws.cell_start, a.r2, a.K,
                       a.src, a.dst, a.edge_capacity, ws.plans, ws.ctr, a.edge_off_out ? a.edge_off_out : ws.edge_off,
                       a.report_out ? a.report_out : ws.report);
}

template <int DP>
int occupancy_blocks(bool sel, bool four) {
    const auto kernel = sel ? (four ? k_search<DP, true, true> : k_search<DP, true, false>)
                            : (four ? k_search<DP, false, true> : k_search<DP, false, false>);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 256;
    return per_cu * cus;
}

}  // namespace

int search_blocks_for(int dpad, bool sel, bool four) {
    switch (dpad) {
        case 4: return occupancy_blocks<4>(sel, four);
        case 8: return occupancy_blocks<8>(sel, four);
        case 12: return occupancy_blocks<12>(sel, four);
        case 16: return occupancy_blocks<16>(sel, four);
        case 24: return occupancy_blocks<24>(sel, four);
        case 32: return occupancy_blocks<32>(sel, four);
        case 48: return occupancy_blocks<48>(sel, four);
        default: return occupancy_blocks<64>(sel, four);
    }
}

hipError_t enqueue_build(const LaunchArgs &a, const Workspace &ws) {
    auto mark = [&](int stage) {
        if (a.events) (void)hipEventRecord(a.events[stage], a.stream);
    };
    const int vec4 = a.vec4;
    const long long kb = (static_cast<long long>(a.max_n) + kKeysSpan - 1) / kKeysSpan;
    const int gkeys = static_cast<int>(kb < 1 ? 1 : kb);
    Dims dd;
    for (int p = 0; p < kMaxAxes; ++p) dd.c[p] = p < a.axes ? a.dims[p] : -1;
    mark(0);
    if (a.bin_span)
        hipLaunchKernelGGL(k_bounds, dim3(a.bounds_blocks, a.n_events), dim3(kBlock), 0, a.stream, a.d, dd, vec4,
                           ws.ev, a.ev0, a.ev_from_arg, ws.part, crowd_counts(ws), crowd_at(ws.rows, a.tile_points) + 1,
                           crowd_sums(ws), a.n_events, ws.ctr);
    else
        hipLaunchKernelGGL(k_bounds, dim3(a.bounds_blocks, a.n_events), dim3(kBlock), 0, a.stream, a.d, dd, vec4,
                           ws.ev, a.ev0, a.ev_from_arg, ws.part, ws.cell_count, ws.cells, ws.sums_cells,
                           ws.tiles_cells_n, ws.ctr);
    mark(1);
    if (a.bin_span) {
        const int flat = flat_grid(a, ws.rows) ? a.n_events : 0;
        const dim3 grid = flat ? dim3(static_cast<unsigned int>(blocks_before(ws.rows, a.n_events, a.bin_span, 1) + 1))
                               : dim3(static_cast<unsigned int>(a.max_n < 1 ? 1 : (a.max_n + a.bin_span - 1) / a.bin_span),
                                      a.n_events);
        if (a.bin_span == kKeysBlock)
            hipLaunchKernelGGL(k_bin<1>, grid, dim3(kKeysBlock), 0, a.stream, a.d, dd, a.axes, a.r, a.cell_div, a.tile_points,
                               ws.ev, a.ev0, a.ev_from_arg, flat, ws.part, a.bounds_blocks, ws.plans, ws.ctr,
                               bin_ents(ws), bin_table(ws), crowd_counts(ws), crowd_sums(ws));
        else
            hipLaunchKernelGGL(k_bin<2>, grid, dim3(kKeysBlock), 0, a.stream, a.d, dd, a.axes, a.r, a.cell_div, a.tile_points,
                               ws.ev, a.ev0, a.ev_from_arg, flat, ws.part, a.bounds_blocks, ws.plans, ws.ctr,
                               bin_ents(ws), bin_table(ws), crowd_counts(ws), crowd_sums(ws));
        mark(2);  // there is no stage 2: stage 3 begins here
    } else {
        hipLaunchKernelGGL(k_keys, dim3(gkeys, a.n_events), dim3(kKeysBlock), 0, a.stream, a.d, dd, a.axes,
                           a.r, a.cell_div, ws.ev, a.ev0, a.ev_from_arg, ws.part, a.bounds_blocks, ws.plans, ws.ctr,
                           ws.pcell, ws.rank, ws.cell_count, ws.sums_cells);
        mark(2);
        hipLaunchKernelGGL(k_scan_cells, dim3(ws.tiles_cells_n), dim3(kBlock), 0, a.stream, ws.cell_count, ws.cells,
                           ws.sums_cells, ws.tiles_cells_n, ws.cell_start, ws.wave_start,
                           a.search_blocks * kWaves, ws.rows, ws.claims);
        mark(3);
    }
    switch (a.dpad) {
        case 4: launch_rows<4>(a, ws, vec4); break;
        case 8: launch_rows<8>(a, ws, vec4); break;
        case 12: launch_rows<12>(a, ws, vec4); break;
        case 16: launch_rows<16>(a, ws, vec4); break;
        case 24: launch_rows<24>(a, ws, vec4); break;
        case 32: launch_rows<32>(a, ws, vec4); break;
        case 48: launch_rows<48>(a, ws, vec4); break;
        default: launch_rows<64>(a, ws, vec4); break;
    }
    mark(7);
    return hipGetLastError();
}

}  // namespace frnn
