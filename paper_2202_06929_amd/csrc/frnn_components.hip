// Track labeling on the FRNN edge list: weakly connected components of the kept
// edges, every vertex labeled with the smallest vertex id of its component
// (paper, Section 2: the edges whose score passes a threshold are kept and each
// weakly connected component is a track candidate; Section 3.2: the labeling
// runs on the edge list that already exists).
//
// Lock-free union-find on a parent array (one 32-bit entry per vertex):
//   k_cc_init     parent[v] = v
//   k_cc_minhook  each source hooked under its smallest neighbour (see there), so
//                 that clusters whose vertices all neighbour their smallest vertex
//                 are stars before the next pass
//   k_cc_hook     one lane per kept edge: find both roots (plain reads: the only
//                 writes of this kernel are the hooks, device-scope atomics that are
//                 performed beyond the per-XCD caches and cost memory traffic), hook
//                 the larger root under the smaller one with a compare-and-swap if a
//                 device-scope load still finds it a root, retry from the new roots
//                 if another thread hooked it first
//   k_cc_label    label[v] = root of v (path halving); counts the roots; the last
//                 workgroup writes the component count and the status
// Parent pointers only ever point to smaller ids (hooks go from the larger root
// to the smaller, halving jumps to an ancestor), so there are no cycles and every
// find ends.  When all edges are done each component is one tree, and its root is
// its smallest vertex: that vertex's parent cannot be smaller, so it is a root.
// Finds read the parent array with ordinary (cached) loads: a stale entry is still
// an ancestor, because entries only ever move up the tree, so a find returns a
// vertex of the right tree, perhaps not its current root.  Equal results therefore
// prove two vertices share a tree.  Hooks are device-scope compare-and-swaps on
// the presumed root; where it is none any more its current parent, a strictly
// smaller id, is known, and the hook resumes from there, so every retry makes
// progress on fresh data.  Path-halving stores (labeling pass) are device-scope
// atomic stores.

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <atomic>

#include "frnn.h"
#include "frnn_internal.h"

namespace {

constexpr int kCcBlock = 256;
// Rounds of the hook loop per edge before the call reports an internal error.  A
// round repeats only after another thread merged one of the two trees, so a
// correct run needs at most one round per merge; the bound is a safety net.
constexpr unsigned int kMaxHookRounds = 1u << 20;

struct CcState {
    unsigned int status;             // bit 0: endpoint out of range; bit 1: hook bound reached
    unsigned int pad;
    // Labeling workgroups done (bits 44..63) and roots counted so far (bits 0..43),
    // one word so that a single atomic add both counts and tells the last workgroup.
    unsigned long long done_roots;
};

constexpr int kRootBits = 44;
constexpr unsigned long long kRootMask = (1ull << kRootBits) - 1;

__device__ __forceinline__ long long status_code(unsigned int s) {
    return (s & 1u) ? FRNN_ERR_ARG : ((s & 2u) ? FRNN_ERR_HIP : FRNN_OK);
}

__device__ __forceinline__ unsigned int ld(const unsigned int *p) { return *p; }

__device__ __forceinline__ void st(unsigned int *p, unsigned int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of x, halving the path on the way (x is pointed at its grandparent).
__device__ unsigned int cc_find(unsigned int *parent, unsigned int x) {
    for (;;) {
        const unsigned int p = ld(parent + x);
        if (p == x) return x;
        const unsigned int gp = ld(parent + p);
        if (gp == p) return p;
        st(parent + x, gp);
        x = gp;
    }
}

// Root of x by plain reads (no path halving).
__device__ __forceinline__ unsigned int cc_root(unsigned int *parent, unsigned int x) {
    for (;;) {
        const unsigned int p = ld(parent + x);
        if (p == x) return x;
        x = p;
    }
}

// Roots of x and y by plain reads, the two walks interleaved so that their loads
// overlap.
__device__ void cc_find2(unsigned int *parent, unsigned int &x, unsigned int &y) {
    bool dx = false, dy = false;
    while (!(dx && dy)) {
        const unsigned int px = dx ? x : ld(parent + x);
        const unsigned int py = dy ? y : ld(parent + y);
        dx = dx || px == x;
        dy = dy || py == y;
        const unsigned int gx = dx ? x : ld(parent + px);
        const unsigned int gy = dy ? y : ld(parent + py);
        if (!dx) {
            if (gx == px) {
                x = px;
                dx = true;
            } else {
                x = gx;
            }
        }
        if (!dy) {
            if (gy == py) {
                y = py;
                dy = true;
            } else {
                y = gy;
            }
        }
    }
}

// Joins the trees of u and v: hooks the larger root under the smaller with a
// compare-and-swap.  u and v need not be roots: where the larger one is none any more, its
// current parent is a strictly smaller id, and the join resumes from that one's root, so
// the larger of the pair decreases every round.  A device-scope load tells first whether
// it is still a root: most are not where many edges join the same trees, and swaps of one
// address wait for each other (1M edges of a random graph over 200,000 vertices, whole
// calls: 1,020 to 1,050 us with the swap alone, 220 to 235 with the load before it, four
// edges a lane in both; the 120k-point event's graph 44.2 and 42.6).
__device__ void cc_union(unsigned int *parent, unsigned int u, unsigned int v, CcState *state) {
    for (unsigned int round = 0; u != v; ++round) {
        if (round >= kMaxHookRounds) {
            atomicOr(&state->status, 2u);
            return;
        }
        const unsigned int hi = u > v ? u : v, lo = u > v ? v : u;
        unsigned int now = __hip_atomic_load(parent + hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (now == hi && __hip_atomic_compare_exchange_strong(parent + hi, &now, lo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT))
            return;
        if (now == lo) return;  // joined meanwhile
        u = cc_root(parent, now);
        v = lo;
    }
}

__global__ __launch_bounds__(kCcBlock) void k_cc_init(unsigned int *parent, long long n, CcState *state) {
    const long long stride = static_cast<long long>(gridDim.x) * kCcBlock;
    for (long long v = static_cast<long long>(blockIdx.x) * kCcBlock + threadIdx.x; v < n; v += stride)
        parent[v] = static_cast<unsigned int>(v);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        CcState z = {};
        *state = z;
    }
}

// Hooks each edge's larger endpoint under its smallest neighbour first, so that a
// cluster whose vertices all neighbour its smallest vertex (the FRNN graph of a
// track: its points lie within r of one another) is a star before the union-find
// pass, which then finds equal roots for its edges and swaps nothing.  Lanes of a
// wave that share a source (edges come grouped by source) take the minimum of their
// targets, the first one where targets ascend and else by a segmented reduction, and
// one lane per source does a device-scope atomicMin on the source's parent.  The parent
// array then still points only to smaller ids and every entry to a neighbour or itself:
// each vertex is hooked at most under one neighbour, a valid union of two trees, as every
// vertex is still a root before this pass.  Whatever this pass leaves unjoined, the
// union-find pass joins.
__global__ __launch_bounds__(kCcBlock) void k_cc_minhook(const long long *__restrict__ src,
                                                         const long long *__restrict__ dst, long long n_edges,
                                                         long long n, const float *__restrict__ scores,
                                                         float threshold, unsigned int *parent) {
    constexpr unsigned int kNone = 0xffffffffu;  // past the end or out of range (reported by the hook pass)
    const int lane = static_cast<int>(threadIdx.x & 63u);
    const long long stride = static_cast<long long>(gridDim.x) * kCcBlock;
    const unsigned long long below = (1ull << lane) - 1ull;
    // Wave-aligned bases, so that every lane of a wave takes the same trip count.
    for (long long e0 = static_cast<long long>(blockIdx.x) * kCcBlock + (threadIdx.x & ~63u); e0 < n_edges;
         e0 += stride) {
        const long long e = e0 + lane;
        const bool in = e < n_edges;
        const long long x = in ? src[e] : -1, y = in ? dst[e] : -1;
        const bool ok = x >= 0 && x < n && y >= 0 && y < n;
        const unsigned int a = ok ? static_cast<unsigned int>(x) : kNone;
        const unsigned int t = ok ? static_cast<unsigned int>(y) : kNone;
        const bool kept = ok && !(scores && !(scores[e] > threshold));
        const unsigned int a_prev = static_cast<unsigned int>(__shfl_up(static_cast<int>(a), 1));
        const unsigned int t_prev = static_cast<unsigned int>(__shfl_up(static_cast<int>(t), 1));
        const bool head = lane == 0 || a_prev != a;
        if (__builtin_amdgcn_ballot_w64(!head && t_prev > t) == 0ull) {
            // Targets ascend within every source, as in the graph builder's lists: a
            // source's smallest kept target is its first.
            const unsigned long long heads = __builtin_amdgcn_ballot_w64(head);
            const unsigned long long keeps = __builtin_amdgcn_ballot_w64(kept);
            const unsigned long long run = ~0ull << (63 - __builtin_clzll(heads & (below | (1ull << lane))));
            if (kept && (keeps & below & run) == 0ull && t < a) atomicMin(parent + a, t);
            continue;
        }
        // Minimum over the lanes at or after this one with the same source.
        unsigned int m = kept ? t : kNone;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int a2 = static_cast<unsigned int>(__shfl_down(static_cast<int>(a), o));
            const unsigned int m2 = static_cast<unsigned int>(__shfl_down(static_cast<int>(m), o));
            if (lane + o < 64 && a2 == a && m2 < m) m = m2;
        }
        if (head && a != kNone && m < a) atomicMin(parent + a, m);
    }
}

// One edge per lane.  Most edges' endpoints have the same parent (after the min-neighbour
// pass) and are done; the others find their roots and join them.  What the pass waits for
// is its chain of round trips and its swaps, so as many edges as fit are in flight at once
// (four per lane in turn: a 120k-point event's graph of 1.06M edges 42.6 us a call
// against 41.1, scored 52.7 and 48.5).  Joining lanes that follow each other with the same
// two trees, as a source's edges do, leave the join to the first of them (1M edges inside
// clusters of ten vertices 54.1 us if only lanes side by side do, 47.5 so).
//
// Where a lane's smaller root is the larger root of the joining lane before or after it (a
// path's edges in either direction), hooking each under the next would build a tree as
// deep as the path, which the labeling pass then climbs: such lanes hook under the end of
// their chain in the wave instead, found by doubling.  Every pair is still joined: each
// lane of a chain joins its larger root with the chain's end, and so with the root it
// would have hooked under, which is the next lane's larger root.  A path of 200,000
// vertices in rising order takes 58 us (890 without), in falling order 57 (890), one of
// 100 vertices 25.6 (31.6).
//
// No order of the edges is singled out: 1M edges to random vertices take 175 us sorted by
// their source and 205 unsorted.  (Edges queued per wave and joined 64 at a time from the
// queue, with the swap alone: 1,540 and 1,040 to 1,160.)
__global__ __launch_bounds__(kCcBlock) void k_cc_hook(const long long *__restrict__ src,
                                                      const long long *__restrict__ dst, long long n_edges,
                                                      long long n, const float *__restrict__ scores,
                                                      float threshold, unsigned int *parent, CcState *state) {
    const int lane = static_cast<int>(threadIdx.x & 63u);
    const long long stride = static_cast<long long>(gridDim.x) * kCcBlock;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (long long e0 = static_cast<long long>(blockIdx.x) * kCcBlock + (threadIdx.x & ~63u); e0 < n_edges;
         e0 += stride) {
        const long long e = e0 + lane;
        bool act = e < n_edges && !(scores && !(scores[e] > threshold));
        const long long a = act ? src[e] : 0, b = act ? dst[e] : 0;
        if (act && (a < 0 || a >= n || b < 0 || b >= n)) {
            atomicOr(&state->status, 1u);
            act = false;
        }
        unsigned int x = act ? ld(parent + a) : 0u, y = act ? ld(parent + b) : 0u;
        if (x != y) cc_find2(parent, x, y);
        const unsigned int hi = max(x, y);
        unsigned int lo = min(x, y);
        const bool join = hi != lo;
        const unsigned long long joins = __builtin_amdgcn_ballot_w64(join);
        if (joins == 0ull) continue;
        // The joining lanes beside this one (itself at the ends).
        const unsigned long long lower = joins & below, higher = joins & ~below & ~(1ull << lane);
        const int before = lower ? 63 - __builtin_clzll(lower) : lane;
        const int after = higher ? __builtin_ctzll(higher) : lane;
        const unsigned int hi_before = static_cast<unsigned int>(__shfl(static_cast<int>(hi), before));
        const unsigned int lo_before = static_cast<unsigned int>(__shfl(static_cast<int>(lo), before));
        const unsigned int hi_after = static_cast<unsigned int>(__shfl(static_cast<int>(hi), after));
        const bool repeated = before != lane && hi_before == hi && lo_before == lo;
        const bool up = join && hi_before == lo;
        const bool down = join && hi_after == lo;
        if (__builtin_amdgcn_ballot_w64(up || down) != 0ull) {
            int next = up ? before : (down ? after : lane);  // larger roots fall along a chain: it ends
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                lo = static_cast<unsigned int>(__shfl(static_cast<int>(lo), next));
                next = __shfl(next, next);
            }
        }
        if (join && !repeated) cc_union(parent, hi, lo, state);
    }
}

// Vertices per lane in the label pass: their loads are all issued before any is used, so a
// wave keeps several round trips in flight.
constexpr int kPerLane = 4;

// Labels every vertex with its root and counts the roots; the last workgroup to
// finish writes the caller's result [n_components, status].
__global__ __launch_bounds__(kCcBlock) void k_cc_label(unsigned int *parent, long long n, long long *labels,
                                                       CcState *state, long long *result) {
    __shared__ unsigned long long part[kCcBlock / 64];
    const long long span = static_cast<long long>(kCcBlock) * kPerLane;
    const long long stride = static_cast<long long>(gridDim.x) * span;
    unsigned long long roots = 0;
    for (long long v0 = static_cast<long long>(blockIdx.x) * span + threadIdx.x; v0 < n; v0 += stride) {
        // Parents and grandparents of kPerLane vertices requested together; most
        // trees are one or two levels deep by now.
        unsigned int p[kPerLane], g[kPerLane];
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const long long v = v0 + static_cast<long long>(kCcBlock) * j;
            p[j] = v < n ? ld(parent + v) : 0u;
        }
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) g[j] = ld(parent + p[j]);
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const long long v = v0 + static_cast<long long>(kCcBlock) * j;
            if (v >= n) continue;
            const unsigned int r = g[j] == p[j] ? p[j] : cc_find(parent, g[j]);
            labels[v] = static_cast<long long>(r);
            roots += r == static_cast<unsigned int>(v) ? 1ull : 0ull;
        }
    }
    for (int o = 32; o > 0; o >>= 1) roots += __shfl_xor(roots, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = roots;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < kCcBlock / 64; ++w) t += part[w];
        const unsigned long long old = atomicAdd(&state->done_roots, (1ull << kRootBits) | t);
        if ((old >> kRootBits) == gridDim.x - 1u) {
            result[0] = static_cast<long long>((old & kRootMask) + t);
            result[1] = status_code(state->status);
        }
    }
}

// The caller's device result [n_components, status] of a graph without vertices.
__global__ void k_cc_result(const CcState *state, long long *result) {
    result[0] = 0;
    result[1] = status_code(state->status);
}

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

int grid_for(long long items) {
    const long long b = (items + kCcBlock - 1) / kCcBlock;
    return static_cast<int>(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

int check(const int64_t *src, const int64_t *dst, int64_t n_edges, int64_t n_vertices, void *workspace,
          size_t workspace_bytes, int64_t *labels) {
    if (n_edges < 0 || n_vertices < 0) return FRNN_ERR_ARG;
    if (n_vertices >= (int64_t{1} << 31)) return FRNN_ERR_UNSUPPORTED;
    if (n_edges > 0 && (!src || !dst)) return FRNN_ERR_ARG;
    if (n_vertices > 0 && !labels) return FRNN_ERR_ARG;
    if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return FRNN_ERR_ARG;
    if (workspace_bytes < frnn_components_workspace_bytes(n_vertices)) return FRNN_ERR_WORKSPACE;
    return FRNN_OK;
}

int enqueue(const int64_t *src, const int64_t *dst, int64_t n_edges, int64_t n_vertices, const float *scores,
            float threshold, void *workspace, int64_t *labels, int64_t *result_device, hipStream_t s) {
    CcState *state = static_cast<CcState *>(workspace);
    unsigned int *parent = reinterpret_cast<unsigned int *>(static_cast<char *>(workspace) + 256);
    const long long n = n_vertices;
    hipLaunchKernelGGL(k_cc_init, dim3(grid_for(n)), dim3(kCcBlock), 0, s, parent, n, state);
    if (n_edges > 0)
        hipLaunchKernelGGL(k_cc_minhook, dim3(grid_for(n_edges)), dim3(kCcBlock), 0, s,
                           reinterpret_cast<const long long *>(src), reinterpret_cast<const long long *>(dst),
                           static_cast<long long>(n_edges), n, scores, threshold, parent);
    if (n_edges > 0)
        hipLaunchKernelGGL(k_cc_hook, dim3(grid_for(n_edges)), dim3(kCcBlock), 0, s,
                           reinterpret_cast<const long long *>(src), reinterpret_cast<const long long *>(dst),
                           static_cast<long long>(n_edges), n, scores, threshold, parent, state);
    if (n > 0)
        hipLaunchKernelGGL(k_cc_label, dim3(grid_for((n + kPerLane - 1) / kPerLane)), dim3(kCcBlock), 0, s, parent, n,
                           reinterpret_cast<long long *>(labels), state, reinterpret_cast<long long *>(result_device));
    else
        hipLaunchKernelGGL(k_cc_result, dim3(1), dim3(1), 0, s, state, reinterpret_cast<long long *>(result_device));
    return hipGetLastError() == hipSuccess ? FRNN_OK : FRNN_ERR_HIP;
}

thread_local frnn::MappedResult t_result;  // [n_components, status]

}  // namespace

extern "C" size_t frnn_components_workspace_bytes(int64_t n_vertices) {
    if (n_vertices < 0 || n_vertices >= (int64_t{1} << 31)) return 0;
    // state, a 16-byte device result, then the parent array
    return 256 + align256(sizeof(unsigned int) * static_cast<size_t>(n_vertices)) + 256;
}

extern "C" int frnn_components_async(const int64_t *src, const int64_t *dst, int64_t n_edges, int64_t n_vertices,
                                     const float *scores, float threshold, void *workspace, size_t workspace_bytes,
                                     int64_t *labels, int64_t *result_device, void *stream) {
    const int st = check(src, dst, n_edges, n_vertices, workspace, workspace_bytes, labels);
    if (st != FRNN_OK) return st;
    if (!result_device) return FRNN_ERR_ARG;
    return enqueue(src, dst, n_edges, n_vertices, scores, threshold, workspace, labels, result_device,
                   static_cast<hipStream_t>(stream));
}

extern "C" int frnn_components(const int64_t *src, const int64_t *dst, int64_t n_edges, int64_t n_vertices,
                               const float *scores, float threshold, void *workspace, size_t workspace_bytes,
                               int64_t *labels, int64_t *n_components, void *stream) {
    const int st = check(src, dst, n_edges, n_vertices, workspace, workspace_bytes, labels);
    if (st != FRNN_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // The last kernel writes the result straight into pinned host memory when the runtime
    // maps it for the device (a copy enqueued behind the kernels took several us);
    // otherwise it is copied back.
    if (!t_result.ready(2 * sizeof(long long))) return FRNN_ERR_HIP;
    long long *const result = static_cast<long long *>(t_result.host);
    int64_t *result_device = t_result.dev ? static_cast<int64_t *>(t_result.dev)
                                          : reinterpret_cast<int64_t *>(
                                                static_cast<char *>(workspace) + 256 +
                                                align256(sizeof(unsigned int) * static_cast<size_t>(n_vertices)));
    result[1] = FRNN_ERR_HIP;  // until the result arrives
    const int e = enqueue(src, dst, n_edges, n_vertices, scores, threshold, workspace, labels, result_device, s);
    if (e != FRNN_OK) return e;
    if (!t_result.dev &&
        hipMemcpyAsync(result, result_device, 2 * sizeof(long long), hipMemcpyDeviceToHost, s) != hipSuccess)
        return FRNN_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return FRNN_ERR_HIP;
    std::atomic_thread_fence(std::memory_order_acquire);
    if (n_components) *n_components = result[0];
    return static_cast<int>(result[1]);
}
