// ustd_kernels.hip -- gfx950 kernels of the UST estimator of diag(L^+)
// (Angriman, Predari, van der Grinten, Meyerhenke, ESA 2020).
//
//   graph set-up   : int32 row pointers, device CSR validation, max-degree pivot,
//                    level-synchronous BFS with the minimum-ID parent rule (tree B_u)
//   sampling       : Wilson's algorithm, one wavefront per tree, speculative walks with
//                    an in-order commit that reproduces the sequential algorithm exactly
//   tree records   : parent and nearest marked ancestor per vertex (replacing the DFS
//                    timestamps of Algorithm 2); of the caller's own trees by pointer jumping
//   aggregation    : Algorithm 2, thread per vertex over a chunk of resident trees
//   solve          : Jacobi-PCG on the pivot column (FP64, or FP32 inner + FP64 outer)
//   combine        : Eq. diag-comp in FP64
#include "ustd_kernels.hpp"

#include <algorithm>
#include <climits>
#include <type_traits>

namespace ustd {

// ======================================================================================
// graph set-up
// ======================================================================================
__global__ void col_to_u16_kernel(long long nnz, const int *__restrict__ col, unsigned short *__restrict__ col16) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nnz) col16[e] = (unsigned short)col[e];
}

__global__ void rp_to_i32_kernel(int n, const long long *__restrict__ rp64, int *__restrict__ rp32) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v <= n) rp32[v] = (int)rp64[v];
}

// Structural checks of the input CSR (Section "Problem Description and Notation": simple,
// undirected): row bounds, ascending rows (no duplicates), no self-loops, symmetry.
// Connectivity is checked after the BFS.  err receives a bit per failure class.
__global__ void validate_kernel(int n, long long nnz, const long long *__restrict__ rp64,
                                const int *__restrict__ col, int *__restrict__ err) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v == 0 && (rp64[0] != 0 || rp64[n] != nnz)) atomicOr(err, 1);
    if (v >= n) return;
    const long long lo = rp64[v], hi = rp64[v + 1];
    if (hi < lo || lo < 0 || hi > nnz) { atomicOr(err, 1); return; }
    if (hi == lo) { atomicOr(err, 16); return; }  // isolated vertex
    for (long long e = lo; e < hi; ++e) {
        const int w = col[e];
        if (w < 0 || w >= n) { atomicOr(err, 2); return; }
        if (w == v) { atomicOr(err, 4); return; }
        if (e > lo && col[e - 1] >= w) { atomicOr(err, 2); return; }
        long long a = rp64[w], b = rp64[w + 1];
        bool found = false;
        while (a < b) {
            const long long mid = a + (b - a) / 2;
            const int c = col[mid];
            if (c == v) { found = true; break; }
            if (c < v) a = mid + 1; else b = mid;
        }
        if (!found) { atomicOr(err, 8); return; }
    }
}

// Maximum-degree vertex, smallest ID on ties: max of (deg << 32 | ~id).
__global__ void argmax_degree_kernel(int n, const int *__restrict__ rp, unsigned long long *__restrict__ best) {
    unsigned long long key = 0;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const unsigned long long deg = (unsigned long long)(rp[v + 1] - rp[v]);
        const unsigned long long k = (deg << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)v);
        key = k > key ? k : key;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const unsigned long long o = __shfl_xor(key, d, 64);
        key = o > key ? o : key;
    }
    if (lane_id() == 0) atomicMax(best, key);
}

// Pivot by repeated BFS sweeps (engineering appendix): after each BFS, bound[v] = max(bound[v],
// dist[v]) (bound = dist after the first) and the farthest vertex, largest distance then
// smallest ID, as a packed key; at the end the vertex of smallest bound, then smallest ID.
__global__ void sweep_update_kernel(int n, const int *__restrict__ dist, int *__restrict__ bound, int first,
                                    unsigned long long *__restrict__ far) {
    unsigned long long key = 0;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const int d = dist[v];
        bound[v] = first ? d : max(bound[v], d);
        const unsigned long long k = ((unsigned long long)(unsigned)d << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)v);
        key = k > key ? k : key;
    }
#pragma unroll
    for (int dd = 32; dd > 0; dd >>= 1) {
        const unsigned long long o = __shfl_xor(key, dd, 64);
        key = o > key ? o : key;
    }
    if (lane_id() == 0) atomicMax(far, key);
}
__global__ void argmin_bound_kernel(int n, const int *__restrict__ bound, unsigned long long *__restrict__ best) {
    unsigned long long key = 0;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const unsigned long long k = ((unsigned long long)(0x7FFFFFFFu - (unsigned)bound[v]) << 32) |
                                     (unsigned long long)(0xFFFFFFFFu - (unsigned)v);
        key = k > key ? k : key;
    }
#pragma unroll
    for (int dd = 32; dd > 0; dd >>= 1) {
        const unsigned long long o = __shfl_xor(key, dd, 64);
        key = o > key ? o : key;
    }
    if (lane_id() == 0) atomicMax(best, key);
}

__global__ void bfs_init_kernel(int n, int u, int *__restrict__ dist, int *__restrict__ parB) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) {
        dist[v] = (v == u) ? 0 : INT_MAX;
        parB[v] = (v == u) ? -1 : INT_MAX;
    }
}

// Rows are processed in a degree-balanced way: rows of degree <= heavy_thresh by groups of
// G lanes (one row per group), heavier rows (listed once per graph in ascending order) by a
// whole 256-thread block each.  Grid-stride over a fixed grid, so every reduction order
// depends only on the graph.

// One BFS level: every vertex at distance d offers itself as parent to its unvisited
// neighbours; atomicMin keeps the smallest-ID one among all of them, which is the
// minimum-ID neighbour one level closer to u.  `found` is set if any vertex is reached.
// Levels are queued several at a time: a level whose predecessor reached nothing (*prev == 0)
// has no vertex at distance d and returns at once.
template <int G>
__global__ __launch_bounds__(256) void bfs_level_kernel(RowMap m, int d, int *__restrict__ dist,
                                                        int *__restrict__ parB, int *__restrict__ found,
                                                        const int *__restrict__ prev) {
    if (prev && *prev == 0) return;  // uniform over the grid
    int any = 0;
    auto offer = [&](int v, uint32_t e) {
        const int y = m.col[e];
        const int dy = dist[y];
        if (dy > d) {
            atomicMin(&parB[y], v);
            if (dy != d + 1) dist[y] = d + 1;
            any = 1;
        }
    };
    const int nh = *m.nheavy;
    for (int h = blockIdx.x; h < nh; h += gridDim.x) {
        const int v = m.heavy[h];
        if (dist[v] != d) continue;  // uniform in the block
        row_each(m.rp[v], m.rp[v + 1], threadIdx.x, blockDim.x, [&](uint32_t e) { offer(v, e); });
    }
    const int rows_per_tile = 256 / G;
    const int g = threadIdx.x / G, l = threadIdx.x % G;
    for (int tile = blockIdx.x; tile * rows_per_tile < m.n; tile += gridDim.x) {
        const int v = tile * rows_per_tile + g;
        if (v >= m.n || dist[v] != d) continue;
        const int lo = m.rp[v], hi = m.rp[v + 1];
        if (hi - lo > m.heavy_thresh) continue;
        row_each(lo, hi, l, G, [&](uint32_t e) { offer(v, e); });
    }
    if (__any(any) && lane_id() == 0) atomicOr(found, 1);
}

// heavy-row list, deterministic: per-block counts, one-block scan, ordered writes
__global__ __launch_bounds__(256) void heavy_count_kernel(int n, const int *__restrict__ rp, int thresh,
                                                          int *__restrict__ bcount) {
    __shared__ int sh[5];
    const int v = blockIdx.x * 256 + threadIdx.x;
    const int hv = (v < n && rp[v + 1] - rp[v] > thresh) ? 1 : 0;
    int tot;
    block_incl_scan(hv, &tot, sh);
    if (threadIdx.x == 0) bcount[blockIdx.x] = tot;
}
__global__ __launch_bounds__(256) void heavy_scan_kernel(int nb, int *__restrict__ bcount, int *__restrict__ nheavy) {
    __shared__ int sh[5];
    int carry = 0;
    for (int base = 0; base < nb; base += 256) {
        const int i = base + threadIdx.x;
        const int c = i < nb ? bcount[i] : 0;
        int tot;
        const int incl = block_incl_scan(c, &tot, sh);
        if (i < nb) bcount[i] = carry + incl - c;
        carry += tot;
    }
    if (threadIdx.x == 0) *nheavy = carry;
}
__global__ __launch_bounds__(256) void heavy_write_kernel(int n, const int *__restrict__ rp, int thresh,
                                                          const int *__restrict__ boff, int *__restrict__ heavy) {
    __shared__ int sh[5];
    const int v = blockIdx.x * 256 + threadIdx.x;
    const int hv = (v < n && rp[v + 1] - rp[v] > thresh) ? 1 : 0;
    int tot;
    const int incl = block_incl_scan(hv, &tot, sh);
    if (hv) heavy[boff[blockIdx.x] + incl - 1] = v;
}

__global__ void count_unreached_kernel(int n, const int *__restrict__ dist, int *__restrict__ err) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n && dist[v] == INT_MAX) atomicOr(err, 32);
}

// ======================================================================================
// Wilson sampler (Appendix "Wilson's UST Algorithm"), one 64-lane wavefront per tree.
//
// The sequential definition takes start vertices s = 0..n-1 in ascending order; from each
// s not yet in T it walks until it reaches T and adds the loop erasure of the walk.  Step
// k of the walk from s uses its own Philox word (counter (k/4, s, t)), so the whole walk
// from s is a fixed sequence x_0 = s, x_1, x_2, ... that does not depend on T; T only
// decides where it stops (the first x_i in T) and whether s walks at all.
//
// Lanes therefore run the walks of the next not-in-tree starts speculatively, against the
// tree committed so far, and record their vertices.  Walks are committed strictly in
// start order from a reorder buffer (ROB).  Every commit sees exactly the tree the
// sequential algorithm would see at that start (all earlier starts committed, no later
// one), so it truncates the recorded walk at its first vertex now in T, skips s if s has
// been absorbed meanwhile, and adds the loop erasure (each vertex's successor after its
// last visit).  A recorded walk is always long enough: it stopped at a vertex of an older
// tree, which is still in T.  Three commit paths:
//   - runs of short walks (at most kPathLds steps, kept in LDS) commit as one batch, one
//     lane each.  Nine walks in ten of a small-world graph are a single step, and a run of
//     those needs no test at all: its end is in T for good, and nothing it adds is read by
//     another.  Where the run holds longer walks, the vertices they read beside their start
//     (inner vertices) are tested against the tree, and the batch commits up to the first
//     walk that reads an inner vertex of an earlier one; the starts take part only if an
//     inner vertex lies among the starts in flight, an interval since starts ascend;
//   - longer recorded walks (up to kPath steps) commit cooperatively: a lane per step, the
//     loop erasure by one ballot and one lane read per branch vertex.  A walk that filled its
//     record without reaching the tree it saw takes this path too: the tree has usually
//     grown since, so the record mostly does reach it;
//   - if no recorded vertex is in the tree, one lane turns the record into Next pointers and the
//     wave continues the walk from its last vertex, 64 steps at a time (the sequential algorithm
//     for that start; walk_next).
//
// What bounds it: the latency of a round (allocate, step, commit) times the rounds of a tree, and
// on graphs within the bitmap instruction issue.  A commit round that planned every walk for
// five recorded steps, with a tree test (a global load past the bitmap) per vertex, took half
// of a tree's time.  Without those, with 128 entries, starts from the window's list, the records in
// two arrays and the lone walks of walk_next, a pass went from 1350 to 834 ms (R-MAT scale 22, 8192
// trees), 51.3 to 30.6 ms (R-MAT 19, 777 trees, fewer trees than SIMDs), 8.58 to 5.28 ms (R-MAT 16
// edge counts), 13.1 to 9.06 ms (R-MAT 16), 316 to 198 ms (hyperbolic, 200k vertices) and 5.1 to
// 2.85 ms (32 x 32 grid).
//
// Output per vertex x: the word nba(x) | flags and, where the caller or Algorithm 2 reads it,
// parent_T(x) (see "Marked vertices").
// Launches are persistent: each block takes tree after tree from a queue.
// ======================================================================================
namespace {

template <bool LDS>
constexpr int rob_cap() { return LDS ? kSamplerRobLds : kSamplerRobMax; }
constexpr int kPathLds = 4;    // recorded steps kept in LDS per entry (x_1..x_4)
constexpr int kPath = 250;     // recorded steps per speculative walk (x_1..x_250)
static_assert(kPathLds <= (int)kBatchSteps && kPath <= (int)kWalkDraws, "the bounds of the counters");
static_assert(kPath - kPathLds == kSamplerPathGlobal, "path split");
// reorder-buffer entry states (a byte) besides a finished walk's step count (<= kPath; 0: the
// start was absorbed, nothing to commit):
//   kWalking  - still walking
//   kOverflow - recorded kPath steps without reaching the tree it saw
//   kContinue - an overflowed walk none of whose recorded vertices is in the tree at commit
//   kRewalk   - re-walk from the start (never expected; keeps the commit exact regardless)
constexpr int kWalking = 255, kOverflow = 254, kContinue = 253, kRewalk = 252;
static_assert(kPath < kRewalk, "step counts and states share a byte");
// starts are taken from a list of the free vertices of a window of this many vertices
constexpr int kWin = 256;
static_assert(kWin == 4 * kWave, "four vertices of the window per lane");

// Membership of the tree being built.  Graphs of up to 131072 vertices keep an n-bit
// bitmap in LDS.  Larger graphs use the vertex's own record: its nba field holds kFree until
// the vertex joins the tree (the records are cleared when the tree starts), so a membership
// test reads the line a walk that ends there needs anyway, and joining is the record write
// itself (set() does nothing).  All accesses of a tree's records come from one wavefront,
// whose loads and stores the vector L1 keeps in order.

// entry v of an array of 4-byte entries, one per vertex: a 32-bit offset from a uniform base (4 v <
// 2^32) takes one register and no 64-bit address arithmetic
template <typename T>
__device__ __forceinline__ T &vertex_at(T *base, int v) {
    static_assert(sizeof(T) == 4, "4-byte entries");
    using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return *reinterpret_cast<T *>(reinterpret_cast<C *>(base) + ((uint32_t)v << 2));
}

// the word nba | flags of a vertex, which another lane of the wave may have written
__device__ __forceinline__ int load_nbx(const int *nbw, int v) {
    return __hip_atomic_load(&vertex_at(nbw, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

template <bool LDS>
struct TreeState;

template <>
struct TreeState<true> {
    uint32_t *w;
    // the free vertices among the window's 4 lane .. 4 lane + 3, as 4 bits
    __device__ __forceinline__ uint32_t free4(int base, int lane, int n) const {
        const int v = base + 4 * lane;
        return v < n ? (~w[v >> 5] >> (v & 31)) & 0xFu : 0u;
    }
    __device__ __forceinline__ bool test(int v) const { return (w[v >> 5] >> (v & 31)) & 1u; }
    __device__ __forceinline__ void set(int v) const { atomicOr(w + (v >> 5), 1u << (v & 31)); }
};

template <>
struct TreeState<false> {
    int *nbw;  // the tree's nba words
    __device__ __forceinline__ int nbx(int v) const { return load_nbx(nbw, v); }
    __device__ __forceinline__ uint32_t free4(int base, int lane, int n) const {
        const int v = base + 4 * lane;
        if (v >= n) return 0u;
        const int4 w = *reinterpret_cast<const int4 *>(nbw + v);  // padded to 32 vertices
        return (w.x == kFree ? 1u : 0u) | (w.y == kFree ? 2u : 0u) | (w.z == kFree ? 4u : 0u) | (w.w == kFree ? 8u : 0u);
    }
    __device__ __forceinline__ bool test(int v) const { return nbx(v) != kFree; }
    __device__ __forceinline__ void set(int) const {}
};

// Marked vertices.  Algorithm 2 adds, for v and each edge (a, b) of P(v), +1 when T
// contains a -> b above v and -1 when it contains b -> a above v.  Written per T-ancestor x
// of v (x != u), x contributes only if x lies on P(v) and its tree edge x -> parent_T(x) is
// a B_u edge: +1 when parent_T(x) = parB(x) (that edge of P(v) is traversed forward), -1
// when parB(parent_T(x)) = x and parent_T(x) is on P(v) too (traversed backward).  A
// strict T-ancestor of v on P(v) has a child in B_u, so only vertices that are internal in
// B_u and whose tree edge is a B_u edge ("marked") can contribute.  Each vertex x stores
// nba(x) = nearest marked strict T-ancestor (u if none) and its flags (marked; forward or
// backward edge); cv(x) = x if x is marked, else nba(x), is the nba value of x's children.
// Algorithm 2 then follows the nba chain and decides "on P(v)" with the fixed subtree
// intervals of B_u: a forward x counts if x is on P(v), a backward x if parent_T(x) is.
//
// bflag[x] = (parB(x) + 1) | (1 << 31 if x is internal in B_u), so parB(u) = -1.
__device__ __forceinline__ int bf_parent(int f) { return (int)((unsigned)f & 0x7FFFFFFFu) - 1; }
__device__ __forceinline__ bool bf_internal(int f) { return (unsigned)f >> 31; }
// A record is the word nba(x) | flags and parent_T(x), in two arrays per tree: what a walk that
// ends at x and Algorithm 2 read is the word, so a line holds 32 vertices of it.  Bit 31 = x is
// marked, bit 30 = its tree edge is a forward B_u edge (parent_T(x) = parB(x), marked or not); a
// marked vertex without it has a backward one (parB(parent_T(x)) = x).  Vertex IDs are < 2^30 (a
// connected graph with nnz < 2^31).  cv(x) follows from the word.
constexpr int kMarkBit = (int)0x80000000u;
constexpr int kFwdBit = 0x40000000;
__device__ __forceinline__ int nba_of(int nbx) { return nbx & 0x3FFFFFFF; }
__device__ __forceinline__ int cv_of(int x, int nbx) { return (nbx & kMarkBit) ? x : nba_of(nbx); }
// the flag bits of vertex x (B_u flag word fx) whose tree parent is px (flag word fpx)
__device__ __forceinline__ int mark_bits(int x, int fx, int px, int fpx) {
    const unsigned fwd = px == bf_parent(fx), bwd = bf_parent(fpx) == x;
    const unsigned m = (unsigned)bf_internal(fx) & (fwd | bwd);
    return (int)((m << 31) | (fwd << 30));
}
// The same two bits in the low bits, for a walk step x -> y: the walk records them with y,
// since a vertex kept by the loop erasure has as its tree edge the step after its last visit.
__device__ __forceinline__ int edge_bits(int x, int fx, int y, int fy) {
    return (int)((unsigned)mark_bits(x, fx, y, fy) >> 30);
}
constexpr int kVertexMask = 0x3FFFFFFF;  // a recorded global step is y | edge bits << 30

// The sampler's block is one wavefront.  Its LDS operations execute in issue order, so
// lanes exchange data through LDS with compiler ordering only; a workgroup barrier would
// also wait for every outstanding global load and store.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// Force loaded values into registers here.  A load still in flight when its register is
// reused later makes the compiler wait for the whole in-order memory counter, i.e. for
// every store issued since (the commit phase's record stores).
__device__ __forceinline__ void consume(int a, int b, int c, int d) {
    asm volatile("" ::"v"(a), "v"(b), "v"(c), "v"(d));
}
// Batch-commit conflict tables: two tables of minimum-writer lanes under independent
// hashes; a read conflicts only if both of its slots hold a smaller lane, so collisions
// rarely cut a batch short and a real conflict is never missed.  A batch writes a handful of
// inner vertices into them; together they hold the 256 walk words of a one-lane walk.
constexpr int kHashSlots = 128;

// inclusive prefix sum over the 64 lanes with DPP row shifts and row broadcasts
__device__ __forceinline__ int wave_scan_dpp(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}
// Multiplicative hashes to [0, kHashSlots).  Any hash keeps the commit exact: a collision only
// ends a batch early.  With the tree bitmap in LDS (vertex IDs below 2^17) they take bits
// 16..22 of a 24 x 24-bit product (odd multipliers near 2^24 times the golden ratio and another
// irrational, so consecutive IDs spread over the table): a full-rate v_mul_u32_u24.
template <bool LDS>
__device__ __forceinline__ int hash_slot(int v) {
    if constexpr (LDS) return (int)(__umul24((unsigned)v, 0x9E3779u) >> 16) & (kHashSlots - 1);
    else return (int)(((unsigned)v * 2654435761u) >> 25);
}
template <bool LDS>
__device__ __forceinline__ int hash_slot2(int v) {
    if constexpr (LDS) return (int)((__umul24((unsigned)v, 0xC2B2AFu) + 0x5BD1E9u) >> 16) & (kHashSlots - 1);
    else return (int)(((unsigned)v * 2246822519u + 3266489917u) >> 25);
}
static_assert(kHashSlots == 128, "the hashes give seven bits");

// With the tree state in the records, a table of rounds tells which vertices may have joined T
// lately without a global load: an inner vertex of a walk committed in round r (commits of a round
// follow its steps) leaves r at its slot, so a vertex read as free in round q is still free if
// its slot holds less than q and it is not a start that has been committed since.  A collision
// only costs the load (a long walk's commit leaves a dozen rounds, so 256 slots answered few).
constexpr int kStamps = 1024;
__device__ __forceinline__ int stamp_slot(int v) { return (int)(((unsigned)v * 2654435761u) >> 22); }
static_assert(kStamps == 1024, "the hash gives ten bits");
// Rounds are kept modulo 2^16: whether `stamp` is round r or later.  A walk ends, and a window's
// last start is taken, well within 2^15 rounds (a walk takes at most kPath steps, a window's starts
// pass through the reorder buffer in a few lifetimes of one), so a later stamp is never taken for an
// earlier one; an older stamp that looks later costs a load.
__device__ __forceinline__ bool since(uint16_t stamp, uint32_t r) { return (int16_t)(uint16_t)(stamp - r) >= 0; }

// Neighbour index (0 .. deg-1) of a walk step with word w from the row [r0, r1).  Unit
// weights: floor(w deg / 2^32).  Weighted (Section "Generalizations"): the first j with
// t < C[j], C the row's running conductance sums (cw, taken left to right in FP64) and
// t = (w 2^-32) C[deg-1]; both products are exact or rounded once, so the choice is the
// same on every device, and all-ones weights give floor(w deg / 2^32).
//
// The weighted search starts from a guide entry: bucket i = floor(w deg / 2^32) holds the
// first j with C[j] > t(w_i), w_i the bucket's smallest word.  t is non-decreasing in w, so
// that j never passes the answer, and a forward scan ends on it; buckets are equally wide
// in t, so the scan takes one probe on average for any weights (deg boundaries, deg buckets).
template <bool WT, typename Sums, typename Guide>
__device__ __forceinline__ int step_index(uint32_t w, int r0, int r1, Sums cw, Guide guide) {
    const int bucket = (int)__umulhi(w, (uint32_t)(r1 - r0));
    if constexpr (!WT) {
        return bucket;
    } else {
        const double t = ((double)w * 0x1p-32) * cw[r1 - 1];
        const int last = r1 - r0 - 1;
        int j = guide[r0 + bucket];
        while (j < last && !(t < cw[r0 + j])) ++j;  // t < C[deg-1] for any normal row total
        return j;
    }
}

// ---- the lone walk: the sequential algorithm for one start against the current tree, in two
// parts: a walk that writes Next pointers until it reaches the tree, then the retrace of the
// loop erasure that writes the branch's records.  The walk resumes at step k0 from vertex x0
// (k0 = 0, x0 = s0 for a whole walk; otherwise the Next pointers of steps 0..k0-1 are already
// written).  Every lane calls both.
//
// Next pointers: the parents of the records (a Next becomes the parent when the vertex joins).
struct NextRec {
    int *par;
    __device__ __forceinline__ void set(int x, int y) const { vertex_at(par, x) = y; }
    __device__ __forceinline__ int get(int x) const { return vertex_at(par, x); }
};

__device__ __forceinline__ long long uniform_ll(long long k) {
    const int lo = __builtin_amdgcn_readfirstlane((int)(unsigned long long)k);
    const int hi = __builtin_amdgcn_readfirstlane((int)((unsigned long long)k >> 32));
    return (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Tables that no kernel writes while the sampler runs, read at wave-uniform addresses through the
// scalar cache.
template <typename T>
using scalar_ptr = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ scalar_ptr<T> scalar(const T *p) {
    return (scalar_ptr<T>)(uintptr_t)uniform_ll((long long)(uintptr_t)p);
}
// column of a CSR slot at a wave-uniform address (scalar loads take whole words; nnz is even)
__device__ __forceinline__ int scalar_col(const int *col, int slot) { return scalar(col)[slot]; }
__device__ __forceinline__ int scalar_col(const unsigned short *col, int slot) {
    const uint32_t two = scalar(reinterpret_cast<const uint32_t *>(col))[slot >> 1];
    return (int)((slot & 1) ? two >> 16 : two & 0xFFFFu);
}

// A lone walk is a chain of dependent loads and, on deep graphs, the critical path of the launch
// (160 x 160 grid: 619,000 steps of the slowest tree), so the chain holds nothing but the next
// row: the wave steps through a window of up to 64 steps without looking at the tree, every value
// wave-uniform (a step's word is read from a lane's Philox block by readlane, the row of the
// slot's vertex by one scalar load from `hops`), and keeps the slots, a lane each.  The lanes then
// look up their steps' vertices and test them together; steps past the first tree vertex are
// dropped.  Next pointers: the last step out of a vertex counts, found by comparing all pairs.
//   graph in LDS (GL): the row comes from the packed entries `lhops` {begin, degree << 16}, or
//   from the columns and row pointers where those do not fit;
//   no `hops` (a static scratch did not hold them): from the columns and row pointers, two loads.
// Cycles a step, one lane stepping with the tree test and the store in its chain -> this: rows from
// L2 (160 x 160 grid) 589 -> 227, graph in LDS (32 x 32) 277 -> 161, rows past L2 with the GPU full
// (hyperbolic, n = 200k) 1812 -> 1200.
// Returns the walk's total step count.
template <bool LDS, typename CT, bool WT, bool GL, bool BV, typename Next>
__device__ long long walk_next(const TreeState<LDS> &bits, const Next &next, const int *rp, const CT *col,
                               const unsigned long long *hops, const uint32_t *lhops, const double *cw, const int *guide,
                               uint32_t wkey, int x0, long long k0, uint32_t tlo, uint32_t thi, uint32_t key0,
                               uint32_t key1) {
    const int lane = threadIdx.x;
    long long k = k0;
    int xw = x0;
    int r0 = __builtin_amdgcn_readfirstlane(rp[x0]);  // the row of xw: begin, degree
    int deg = __builtin_amdgcn_readfirstlane(rp[x0 + 1]) - r0;
    if constexpr (GL) {  // LDS answers in vector registers: the chain stays there
        asm volatile("" : "+v"(r0));
        asm volatile("" : "+v"(deg));
    }
    for (;;) {
        // lane i: the words of steps 4 (k / 4 + i) .. + 3; a window is 64 of them from a multiple of 64
        const uint4 ph = philox4x32_10(make_uint4((uint32_t)((k >> 2) + lane), wkey, tlo, thi), key0, key1);
        int j0 = (int)(k & 3);  // first step of the window
        for (int win = 0; win < 4; ++win) {
            int slots = 0;
            auto chase = [&](auto row) {
                auto step = [&](uint32_t w, int j) {
                    const int slot = r0 + step_index<WT>(w, r0, r0 + deg, scalar(cw), scalar(guide));
                    slots = lane == j ? slot : slots;
                    row(slot);
                };
                int j = j0;
                for (; j & 3; ++j) {
                    const uint32_t w = (j & 3) == 1 ? ph.y : ((j & 3) == 2 ? ph.z : ph.w);
                    step((uint32_t)__builtin_amdgcn_readlane((int)w, 16 * win + (j >> 2)), j);
                }
                for (; j < kWave; j += 4) {
                    const int l = 16 * win + (j >> 2);
                    step((uint32_t)__builtin_amdgcn_readlane((int)ph.x, l), j);
                    step((uint32_t)__builtin_amdgcn_readlane((int)ph.y, l), j + 1);
                    step((uint32_t)__builtin_amdgcn_readlane((int)ph.z, l), j + 2);
                    step((uint32_t)__builtin_amdgcn_readlane((int)ph.w, l), j + 3);
                }
            };
            if constexpr (GL) {
                if (lhops)
                    chase([&](int slot) {
                        const uint32_t h = lhops[slot];
                        r0 = (int)(h & 0xFFFFu);
                        deg = (int)(h >> 16);
                    });
                else
                    chase([&](int slot) {
                        const int y = col[slot];
                        r0 = rp[y];
                        deg = rp[y + 1] - r0;
                    });
            } else if ((!LDS && !BV) || hops) {  // past the bitmap always there, but for the block-split graph
                chase([&](int slot) {
                    const unsigned long long h = scalar(hops)[(uint32_t)slot];
                    r0 = (int)(uint32_t)h;
                    deg = (int)(uint32_t)(h >> 32);
                });
            } else {
                chase([&](int slot) {
                    const int y = scalar_col(col, slot);
                    r0 = scalar(rp)[y];
                    deg = scalar(rp)[y + 1] - r0;
                });
            }
            const bool on = lane >= j0;
            const int y = on ? (int)col[slots] : 0;
            const uint64_t in = __ballot(on && bits.test(y));
            const int end = in ? __builtin_ctzll(in) : kWave - 1;  // the last step taken
            int x = __shfl_up(y, 1, kWave);
            if (lane == j0) x = xw;
            const bool taken = on && lane <= end;
            const int xt = taken ? x : -1;
            uint64_t again = 0ull;  // x is left again further on
#pragma unroll
            for (int j = 1; j < kWave; ++j)
                again |= __ballot(xt == __builtin_amdgcn_readlane(xt, j)) & ((1ull << j) - 1ull);
            if (taken && !((again >> lane) & 1ull)) next.set(x, y);
            wave_sync();
            k += end + 1 - j0;
            if (in) return k;
            xw = __builtin_amdgcn_readlane(y, kWave - 1);
            j0 = 0;
        }
    }
}

// Retrace of the loop erasure from s0 along the Next pointers to the tree, and the branch's
// records.  Lane 0 follows the pointers (one dependent load per vertex), up to 256 vertices at a
// time into buf (LDS); the wave then writes their records, a lane each, from the tree's end of
// the piece.  nba of a vertex is the nearest marked one closer to the tree, so the vertices from
// a piece's last marked one on wait for the next piece that has one (or for the tree): they are
// written with a placeholder and completed by lane 0 then.
template <bool LDS, typename Next>
__device__ void retrace(const TreeState<LDS> &bits, const Next &next, int *nbw, int *par, const int *__restrict__ bflag, int u,
                        int s0, int *buf, uint16_t *stamps, uint32_t round) {
    constexpr int kPiece = 2 * kHashSlots;
    const int lane = threadIdx.x;
    int z = s0, pend = -1;  // pend: first vertex whose nba is not known yet
    for (;;) {
        int cnt = 0, fin = 0;
        if (lane == 0) {
            for (;;) {
                const int nz = next.get(z);  // loaded beside the tree test
                if (bits.test(z)) {
                    fin = 1;
                    break;
                }
                if (cnt == kPiece) break;
                buf[cnt++] = z;
                z = nz;
            }
        }
        wave_sync();
        cnt = __builtin_amdgcn_readfirstlane(cnt);
        fin = __builtin_amdgcn_readfirstlane(fin);
        z = __builtin_amdgcn_readfirstlane(z);
        int carry = fin ? cv_of(z, load_nbx(nbw, z)) : -1;
        const int first = cnt ? buf[0] : z;
        int last = -1;  // the piece's last marked vertex
        for (int c = (cnt - 1) >> 6; c >= 0; --c) {  // cnt = 0: no piece
            const int i = c * kWave + lane;
            const bool mine = i < cnt;
            const int v = mine ? buf[i] : 0, nx = mine ? (i + 1 < cnt ? buf[i + 1] : z) : 0;
            const int mb = mine ? mark_bits(v, bflag[v], nx, bflag[nx]) : 0;
            const uint64_t m = __ballot((mb & kMarkBit) != 0);
            const uint64_t above = lane < kWave - 1 ? (m & (~0ull << (lane + 1))) : 0ull;
            const int up = __shfl(v, above ? __builtin_ctzll(above) : 0, kWave);
            const int nba = above ? up : carry;
            if (mine) {
                vertex_at(nbw, v) = (nba >= 0 ? nba : u) | mb;  // the Next pointer is the parent
                bits.set(v);
                if constexpr (!LDS) stamps[stamp_slot(v)] = (uint16_t)round;
            }
            if (m) {
                if (last < 0) last = __builtin_amdgcn_readlane(v, 63 - __builtin_clzll(m));
                carry = __builtin_amdgcn_readlane(v, __builtin_ctzll(m));
            }
        }
        wave_sync();
        if (pend >= 0 && carry >= 0) {
            if (lane == 0)
                for (int w = pend; w != first; w = par[w]) {
                    const int old = load_nbx(nbw, w);
                    vertex_at(nbw, w) = carry | (old & ~kVertexMask);
                }
            pend = -1;
            wave_sync();
        }
        if (fin) return;
        if (last >= 0) pend = last;
        else if (pend < 0) pend = first;
    }
}

}  // namespace

// five waves a SIMD (96 registers): one register more and the compiler drops to four
template <bool LDS, typename CT, bool WT, bool GL = false, bool BV = false>
__global__ __launch_bounds__(64, 5) void wilson_kernel(WilsonArgs a) {
    // Reorder buffer.  Vertex IDs take the column type (16 bits when n <= 65536): 14 bytes an
    // entry, so that with the tree bitmap a block of R-MAT scale 16 fits 18 to a CU at 128
    // entries.  A recorded step keeps the vertex and the step's edge bits (below).
    constexpr int kRobMax = rob_cap<LDS>();
    struct alignas(2 * sizeof(CT)) Ends { CT s, cv; };       // start; chain value of the walk's end
    struct alignas(4 * sizeof(CT)) Steps { CT v[kPathLds]; };  // x_1 .. x_4
    extern __shared__ uint32_t lds_bits[];
    __shared__ Ends rob_e[kRobMax];
    __shared__ Steps rob_p[kRobMax];
    __shared__ uint8_t rob_k[kRobMax];
    __shared__ uint8_t rob_pb[kRobMax];  // edge bits of steps 1..kPathLds, 2 bits each
    __shared__ uint16_t rob_r[LDS ? 1 : kRobMax];  // round of a finished walk's last step (low 16 bits)
    __shared__ alignas(16) int htab[2 * kHashSlots];
    __shared__ uint16_t stamps[LDS ? 1 : kStamps];
    __shared__ uint8_t win[kWin];  // free vertices of the window, as offsets
    int *const hslot = htab;                // first conflict table
    int *const hslot2 = htab + kHashSlots;  // second conflict table; together the record of an
                                            // overflowed walk and a retrace's pieces (then cleared)
    static_assert(kPath + 1 <= 2 * kHashSlots, "a record fits the tables");
    static_assert(kPathLds * 2 <= 8, "edge bits fit rob_pb");

    const int lane = threadIdx.x;
    int *__restrict__ gpath = a.path + (long long)blockIdx.x * kSamplerPathSlot;

    // GL (small graphs, single-graph launches): the row pointers, B_u flags and 16-bit columns
    // are copied into LDS after the tree bitmap, once per block, so that walk steps read LDS
    // instead of the L1/L2; with a.lds_hops also the rows of the lone walk, packed.
    const int *lrp = nullptr, *lbf = nullptr;
    const uint32_t *lhops = nullptr;
    const CT *lcol = nullptr;
    if constexpr (GL) {
        static_assert(LDS && !WT && sizeof(CT) == 2, "graph in LDS: small unweighted graphs");
        const int n0 = a.g.n;
        int *srp = reinterpret_cast<int *>(lds_bits + a.g.nwords);
        int *sbf = srp + n0 + 1;
        const int nnz0 = a.g.rp[n0];
        uint32_t *shop = reinterpret_cast<uint32_t *>(sbf + n0);
        CT *scol = reinterpret_cast<CT *>(shop + (a.lds_hops ? nnz0 : 0));
        const CT *gcol = reinterpret_cast<const CT *>(a.g.colv);
        for (int i = lane; i <= n0; i += kWave) srp[i] = a.g.rp[i];
        for (int i = lane; i < n0; i += kWave) sbf[i] = a.g.bflag[i];
        for (int i = lane; i < nnz0; i += kWave) scol[i] = gcol[i];
        wave_sync();
        if (a.lds_hops) {
            for (int i = lane; i < nnz0; i += kWave) {
                const int y = (int)scol[i];
                shop[i] = (uint32_t)srp[y] | ((uint32_t)(srp[y + 1] - srp[y]) << 16);
            }
            wave_sync();
            lhops = shop;
        }
        lrp = srp;
        lbf = sbf;
        lcol = scol;
    }

    for (;;) {
    // ---------------------------------------------------------------- next tile
    // The barrier keeps the wave together here: without a convergent operation between the
    // lane-0 branch at the end of a tile and the one below, the compiler may join the two and
    // send the other lanes into the next tile alone.
    wave_sync();
    int tile = 0;
    if (lane == 0) tile = atomicAdd(a.queue, 1);
    tile = __builtin_amdgcn_readfirstlane(tile);
    if (tile >= a.ntiles) break;
    WilsonGraph g;
    long long t;
    int *nbw;  // the tree's records: nba words, then parents
    if (a.tiles) {
        const WilsonTile tl = a.tiles[tile];
        g = a.graphs[tl.graph];
        t = tl.tree;
        nbw = a.rec + tl.rec_off;
    } else {
        g = a.g;
        t = a.tree_begin + tile;
        nbw = a.rec + (long long)tile * 2 * g.rec_stride;
    }
    const int n = g.n;
    const int nwords = g.nwords;
    const int rob = min(g.rob, kRobMax);  // power of two
    const int robm = rob - 1;
    const uint32_t tlo = (uint32_t)(unsigned long long)t, thi = (uint32_t)((unsigned long long)t >> 32);
    int *par = nbw + g.rec_stride;  // (Next while walking)
    TreeState<LDS> bits;
    if constexpr (LDS) bits.w = lds_bits;
    else bits.nbw = nbw;
    const NextRec next{par};
    const int *__restrict__ bflag = GL ? lbf : g.bflag;
    const int4 *__restrict__ vrow = g.vrow;
    const int u = g.u;
    const int *__restrict__ rp = GL ? lrp : g.rp;
    const CT *__restrict__ col = GL ? lcol : reinterpret_cast<const CT *>(g.colv);  // int32, or uint16 when n <= 65536
    const double *__restrict__ cw = g.cw;
    const int *__restrict__ guide = g.guide;

    if constexpr (LDS) {
        for (int i = lane; i < nwords; i += kWave) bits.w[i] = 0u;
    } else {
        int4 *w4 = reinterpret_cast<int4 *>(nbw);  // padded to 32 vertices
        for (int i = lane; 4 * i < n; i += kWave) w4[i] = make_int4(kFree, kFree, kFree, kFree);
    }
    for (int i = lane; i < 2 * kHashSlots; i += kWave) htab[i] = kWave;
    if constexpr (!LDS)
        for (int i = lane; i < kStamps; i += kWave) stamps[i] = 0xFFFF;  // before round 0
    wave_sync();
    if constexpr (BV) {  // several roots (one per block of the block-split graph)
        for (int i = lane; i < a.nroots; i += kWave) {
            const int r = a.roots[i];
            bits.set(r);
            nbw[r] = r;
            par[r] = -1;
        }
    } else if (lane == 0) {
        bits.set(u);
        nbw[u] = u;
        par[u] = -1;
    }
    wave_sync();

    int head = 0, tail = 0;               // wave-uniform
    int wend = 0, wpos = 0, wcnt = 0;     // the window is [wend - kWin, wend); list position and length
    uint32_t wround = 0;                  // the round that read the window
    int shi = -1;                         // the last start taken
    int mode = 0;                         // 0 idle, 1 speculative walk
    int my_e = 0, x = 0, s = 0, bkey = 0, k = 0, r0 = 0, r1 = 0, fx = 0, pbits = 0;
    uint4 ph = make_uint4(0, 0, 0, 0);
    int4 vx = make_int4(0, 0, 0, 0);  // tree state in the records: x's entry {row begin, row end, B_u flag, 0}
    uint32_t steps = 0u, draws = 0u;      // walk steps and draws of this lane
    long long wsteps = 0, wdraws = 0;     // and of the wave

    // whether a vertex's parent is written, given the edge bits of its tree edge in the low two
    // bits: always, or where Algorithm 2 may read it (marked by a backward edge)
    const bool all_parents = a.parents != 0;
    auto keeps_parent = [&](int eb) { return all_parents || (eb & 3) == 2; };

    // Marks the pending entries whose start has joined the tree (state 0).  With the LDS bitmap
    // the commit tests the start itself; with the tree state in the records that would be a
    // global load per batch, so the marks are brought up to date after a commit that added an
    // inner vertex among the starts in flight, and a commit trusts them.
    auto remark = [&]() {
        for (int o = 0; o < tail - head; o += kWave) {
            const int e = head + o + lane;
            if (e < tail && bits.test((int)rob_e[e & robm].s)) rob_k[e & robm] = 0;
        }
        wave_sync();
    };

    for (uint32_t round = 0;; ++round) {  // used modulo 2^16 (a large tree takes more than 2^31)
        if constexpr (!LDS) {  // walks whose start has been absorbed end (before their slot is given away)
            if (mode == 1 && rob_k[my_e & robm] == 0) mode = 0;
        }
        // ---------------------------------------------------------------- allocate
        // The idle lane of rank r takes the r-th next vertex of the window's list of free vertices
        // (ascending start order).  The list is built once per window, by a prefix sum over the
        // lanes' four vertices; a vertex that joined the tree since is found by a test here and
        // takes an entry that commits nothing (the sequential algorithm skips it).  Few idle
        // lanes are filled every fourth round only: walks that start together need their Philox
        // block in the same round, so in long-walk phases three rounds of four run without one.
        const uint64_t idle = __ballot(mode == 0);
        const int want = min((int)__popcll(idle), rob - (tail - head));
        if (want > 0 && (4 * want >= min(rob, kWave) || (round & 3) == 0 || head == tail) && (wpos < wcnt || wend < n)) {
            const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(idle >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)idle, 0u));
            int got = 0, mys = 0;
            uint32_t myr = 0;  // the round that read the window of mys
            do {
                if (wpos == wcnt) {
                    if (wend >= n) break;
                    if constexpr (!LDS) {  // never due on a graph within the bitmap
                        if (draws_move(wend)) {
                            wdraws += uniform_ll((long long)wave_sum((unsigned long long)draws));
                            draws = 0u;
                        }
                    }
                    uint32_t fb = bits.free4(wend, lane, n);
                    const int left = n - (wend + 4 * lane);
                    if (left < 4) fb &= left > 0 ? (1u << left) - 1u : 0u;
                    const int incl = wave_scan_dpp(__popc(fb));
                    int at = incl - __popc(fb);
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if ((fb >> b) & 1u) win[at++] = (uint8_t)(4 * lane + b);
                    wcnt = __builtin_amdgcn_readlane(incl, kWave - 1);
                    wpos = 0;
                    wend += kWin;
                    wround = round;
                    wave_sync();
                    continue;
                }
                const int take = min(want - got, wcnt - wpos);
                const int j = rank - got;  // this lane's place in this take
                if (mode == 0 && j >= 0 && j < take) {
                    mys = wend - kWin + (int)win[wpos + j];
                    myr = wround;
                }
                got += take;
                wpos += take;
            } while (got < want);
            const bool mode0 = mode == 0;
            if (mode0 && rank < got) {
                my_e = tail + rank;
                s = mys;
                if constexpr (BV) bkey = a.skey[s];
                x = s;
                k = 0;
                bool gone;  // joined the tree since the window was read
                if constexpr (LDS) {
                    r0 = vertex_at(rp, s);
                    r1 = vertex_at(rp, s + 1);
                    fx = vertex_at(bflag, s);
                    gone = bits.test(s);
                } else {
                    vx = vrow[s];  // in flight until the step's random words are there
                    gone = since(stamps[stamp_slot(s)], myr) && bits.test(s);
                }
                pbits = 0;
                mode = gone ? 0 : 1;
                const int sl = my_e & robm;
                rob_e[sl].s = (CT)s;
                rob_k[sl] = (uint8_t)(gone ? 0 : kWalking);
            }
            if (got > 0) shi = __builtin_amdgcn_readlane(mys, __builtin_ctzll(__ballot(mode0 && rank == got - 1)));
            tail += got;
        }
        if (head == tail && wpos == wcnt && wend >= n) break;
        wave_sync();

        // ---------------------------------------------------------------- one walk step
        if (mode == 1) {
            const int sl = my_e & robm;
            if ((k & 3) == 0)
                ph = philox4x32_10(make_uint4((uint32_t)(k >> 2), (uint32_t)(BV ? bkey : s), tlo, thi), g.key0, g.key1);
            const int q = k & 3;
            const uint32_t w = q == 0 ? ph.x : (q == 1 ? ph.y : (q == 2 ? ph.z : ph.w));
            if constexpr (!LDS) {
                r0 = vx.x;
                r1 = vx.y;
                fx = vx.z;
            }
            const int y = (int)col[r0 + step_index<WT>(w, r0, r1, cw, guide)];
            // y's tree membership, with the chain value when the walk ends here, and its B_u flag.
            // With the tree bitmap in LDS (small graphs, whose compact arrays stay in cache) y's row
            // bounds come along if the walk goes on; else y's entry is loaded at the end, and the
            // flag is needed only where x -> y may be a backward B_u edge (x internal in B_u).
            bool in, gone = false;
            int cvy = 0, fy = 0, ny0 = 0, ny1 = 0;
            if constexpr (LDS) {
                fy = vertex_at(bflag, y);
                in = bits.test(y);
                gone = bits.test(s);  // the start has been absorbed: the walk never counts
                if (in) {
                    cvy = load_nbx(nbw, y);
                } else {
                    ny0 = vertex_at(rp, y);
                    ny1 = vertex_at(rp, y + 1);
                }
            } else {
                cvy = bits.nbx(y);  // membership and chain value in one load
                if (bf_internal(fx)) fy = vertex_at(bflag, y);
                in = cvy != kFree;
            }
            consume(fy, cvy, ny0, ny1);  // no load may stay in flight into the commit phase
            if (in) cvy = cv_of(y, cvy);
            ++k;
            ++draws;
            const int eb = edge_bits(x, fx, y, fy);
            if (k <= kPathLds) {
                rob_p[sl].v[k - 1] = (CT)y;
                pbits |= eb << (2 * (k - 1));
                rob_pb[sl] = (uint8_t)pbits;
            } else {
                gpath[sl * kSamplerPathGlobal + (k - 1 - kPathLds)] = y | (eb << 30);
            }
            if (gone) { rob_k[sl] = 0; mode = 0; }
            else if (in) {
                rob_k[sl] = (uint8_t)k;
                rob_e[sl].cv = (CT)cvy;
                if constexpr (!LDS) rob_r[sl] = (uint16_t)round;
                mode = 0;
            } else if (k == kPath) { rob_k[sl] = (uint8_t)kOverflow; mode = 0; }
            else {
                x = y;
                if constexpr (LDS) {
                    fx = fy;
                    r0 = ny0;
                    r1 = ny1;
                } else {
                    vx = vrow[y];
                }
            }
        }
        wave_sync();

        // ---------------------------------------------------------------- in-order commit
        while (head < tail) {
            const int idx = head + lane;
            const int sl = idx & robm;
            const int sk = idx < tail ? (int)rob_k[sl] : kWalking;
            const uint64_t okm = __ballot(sk <= kPathLds);
            const int r = (~okm == 0ull) ? kWave : __builtin_ctzll(~okm);
            if (r > 0) {
                // Batch commit of the done entries head .. head+r-1, one lane each, all planned
                // against the current tree T0.  Entry j's plan is what the sequential algorithm
                // does unless an earlier entry of the batch adds a vertex j has read.
                const Ends en = rob_e[sl];
                const Steps st = rob_p[sl];
                const int pb = (int)rob_pb[sl];
                const int s0 = (int)en.s;
                int carry = (int)en.cv;
                int K = lane < r ? sk : 0;
                if constexpr (LDS) {
                    if (K > 0 && bits.test(s0)) K = 0;  // absorbed
                }
                const uint64_t multi = __ballot(K >= 2);
                const int x1 = (int)st.v[0];
                if (multi == 0ull) {  // single steps only: no two of them interfere
                    if (K > 0) {
                        vertex_at(nbw, s0) = carry | (int)((unsigned)pb << 30);
                        if (keeps_parent(pb)) vertex_at(par, s0) = x1;
                        bits.set(s0);
                        ++steps;
                    }
                    head += r;
                    wave_sync();
                    continue;
                }
                const int slo = __builtin_amdgcn_readfirstlane(s0);  // the starts in flight: slo .. shi
                const int x2 = (int)st.v[1], x3 = (int)st.v[2], x4 = (int)st.v[3];
                const bool any3 = __ballot(K >= 3) != 0ull, any4 = __ballot(K >= 4) != 0ull;  // uniform
                // truncation at the first vertex in T0, whose chain value is then its own
                int istar = K, ya = K >= 2 ? (K == 2 ? x2 : (K == 3 ? x3 : x4)) : x1;
                {
                    int n1 = kFree, n2 = kFree, n3 = kFree;
                    if constexpr (LDS) {
                        if (K >= 2 && bits.test(x1)) n1 = 0;
                        if (any3 && K >= 3 && bits.test(x2)) n2 = 0;
                        if (any4 && K >= 4 && bits.test(x3)) n3 = 0;
                    } else {
                        // x_j was read free in round fin - (K - j); a load only if it may have joined
                        const int fin = (int)rob_r[sl];
                        auto stale = [&](int v, int r) { return v < slo || since(stamps[stamp_slot(v)], r); };
                        const bool t1 = K >= 2 && stale(x1, fin - K + 1);
                        const bool t2 = any3 && K >= 3 && stale(x2, fin - K + 2);
                        const bool t3 = any4 && K >= 4 && stale(x3, fin - K + 3);
                        if (__ballot(t1 || t2 || t3)) {
                            if (t1) n1 = bits.nbx(x1);
                            if (t2) n2 = bits.nbx(x2);
                            if (t3) n3 = bits.nbx(x3);
                        }
                    }
                    int nt = kFree;
                    if (n3 != kFree) { istar = 3; ya = x3; nt = n3; }
                    if (n2 != kFree) { istar = 2; ya = x2; nt = n2; }
                    if (n1 != kFree) { istar = 1; ya = x1; nt = n1; }
                    if constexpr (LDS) {
                        const bool need = istar < K;  // ya joined T after the walk passed it
                        if (__ballot(need)) {
                            if (need) carry = cv_of(ya, load_nbx(nbw, ya));
                        }
                    } else {
                        if (nt != kFree) carry = cv_of(ya, nt);
                    }
                }
                // loop erasure: keep = positions on the erased branch (neighbours on a walk differ)
                unsigned keep = (1u << istar) - 1u;
                if (any3) {
                    if (istar >= 3 && x2 == s0) keep &= ~3u;
                    if (istar == 4) {
                        if (x3 == s0) keep = 8u;
                        else if (x3 == x1 && x2 != s0) keep = 9u;
                    }
                }
                // an inner vertex (read, not in T0) among the starts in flight?
                bool inr = istar >= 2 && x1 >= slo && x1 <= shi;
                if (any3) inr = inr || (istar >= 3 && x2 >= slo && x2 <= shi) || (istar >= 4 && x3 >= slo && x3 <= shi);
                const bool starts = __ballot(inr) != 0ull;
                int jstar = r;
                if (starts || (multi & (multi - 1)) != 0ull) {
                    auto each = [&](auto f) {  // the vertices this lane reads and may add
                        if (starts && K > 0) f(s0);
                        if (istar >= 2) f(x1);
                        if (any3 && istar >= 3) f(x2);
                        if (any4 && istar >= 4) f(x3);
                    };
                    each([&](int v) {
                        atomicMin(&hslot[hash_slot<LDS>(v)], lane);
                        atomicMin(&hslot2[hash_slot2<LDS>(v)], lane);
                    });
                    wave_sync();
                    bool conflict = false;
                    each([&](int v) {
                        if (hslot[hash_slot<LDS>(v)] < lane && hslot2[hash_slot2<LDS>(v)] < lane) conflict = true;
                    });
                    wave_sync();
                    each([&](int v) {
                        hslot[hash_slot<LDS>(v)] = kWave;
                        hslot2[hash_slot2<LDS>(v)] = kWave;
                    });
                    const uint64_t cm = __ballot(conflict);  // never the head: no lane is below it
                    jstar = cm ? __builtin_ctzll(cm) : r;
                }
                if (K > 0 && lane < jstar) {
                    // a kept x_j is the last visit of its vertex, so its tree edge is the
                    // recorded step x_j -> x_{j+1}, whose edge bits are step j+1's
                    int pv = ya;
                    auto put = [&](int j, int v) {
                        if ((keep >> j) & 1u) {
                            const int mb = (int)((unsigned)(pb >> (2 * j)) << 30);
                            vertex_at(nbw, v) = carry | mb;
                            if (keeps_parent(pb >> (2 * j))) vertex_at(par, v) = pv;
                            bits.set(v);
                            if constexpr (!LDS) {
                                if (j > 0) stamps[stamp_slot(v)] = (uint16_t)round;
                            }
                            carry = mb < 0 ? v : carry;  // v is marked
                            pv = v;
                        }
                    };
                    if (any4) put(3, x3);
                    if (any3) put(2, x2);
                    put(1, x1);
                    put(0, s0);
                    steps += istar;
                }
                head += jstar;
                wave_sync();
                if constexpr (!LDS) {
                    if (__ballot(inr && lane < jstar)) remark();
                }
                continue;
            }
            const int hs = __builtin_amdgcn_readfirstlane(sk);
            if (hs == kWalking) break;
            const int hsl = head & robm;
            const int s0 = __builtin_amdgcn_readfirstlane((int)rob_e[hsl].s);
            if constexpr (LDS) {
                if (bits.test(s0)) {  // absorbed
                    ++head;
                    continue;
                }
            }
            // the head's recorded walk x_0..x_K, kPathLds < K <= kPath (an overflowed walk: its
            // whole record, K = kPath): lane j holds x_{j+64c} and the edge bits of the step into it
            const bool ended = hs <= kPath;  // the walk reached the tree it saw
            const int K = ended ? hs : kPath;
            if (ended && K < kWave) {
                // nearly every long commit (hyperbolic, n = 200k: 8,300 a tree, 13 steps on average):
                // one chunk and, the rounds table permitting, no look at the tree in global memory.
                // With the four-chunk form below for all: hyperbolic 206 ms -> 197, R-MAT 19 trees
                // 31.8 -> 30.9, all edges of R-MAT 16 5.44 -> 5.31
                int xv = -1, xb = 0;
                if (lane > kPathLds && lane <= K) {
                    const int e = gpath[hsl * kSamplerPathGlobal + (lane - 1 - kPathLds)];
                    xb = (int)((unsigned)e >> 30);
                    xv = e & kVertexMask;
                } else if (lane == 0) {
                    xv = s0;
                } else if (lane <= kPathLds) {
                    xv = (int)rob_p[hsl].v[lane - 1];
                    xb = ((int)rob_pb[hsl] >> (2 * (lane - 1))) & 3;
                }
                // the first vertex in T: x_K is; of the others those below s0 (all earlier starts are
                // in T), and with the tree state in the records a load only where one may have joined
                bool in = lane == K;
                if constexpr (LDS) {
                    in = lane >= 1 && lane <= K && bits.test(xv);
                } else {
                    const bool inner = lane >= 1 && lane < K;
                    const bool look = inner && xv >= s0 && since(stamps[stamp_slot(xv)], (int)rob_r[hsl] - K + lane);
                    in = in || (inner && xv < s0);
                    if (__ballot(look)) {
                        if (look) in = bits.test(xv);
                    }
                }
                const int istar = __builtin_ctzll(__ballot(in));
                const int ya = __builtin_amdgcn_readlane(xv, istar);
                int carry = (int)rob_e[hsl].cv;
                if (istar < K) carry = cv_of(ya, load_nbx(nbw, ya));
                // loop erasure: from b, jump past b's last visit before istar
                const uint64_t before = (1ull << istar) - 1ull;
                uint64_t kept = 0ull;
                int q = 0;
                do {
                    const uint64_t mm = __ballot(xv == __builtin_amdgcn_readlane(xv, q)) & before;  // holds q
                    q = 63 - __builtin_clzll(mm);
                    kept |= 1ull << q;
                    ++q;
                } while (q < istar);
                const int nx = __shfl_down(xv, 1, kWave), nb = __shfl_down(xb, 1, kWave);
                const bool mine = (kept >> lane) & 1ull;
                const uint64_t m = __ballot(mine && (nb & 2));
                const uint64_t above = lane < kWave - 1 ? (m & (~0ull << (lane + 1))) : 0ull;
                const int up = __shfl(xv, above ? __builtin_ctzll(above) : 0, kWave);
                if (mine) {
                    vertex_at(nbw, xv) = (above ? up : carry) | (nb << 30);
                    if (keeps_parent(nb)) vertex_at(par, xv) = nx;
                    bits.set(xv);
                    if constexpr (!LDS) stamps[stamp_slot(xv)] = (uint16_t)round;
                }
                steps += long_walk_lane<LDS>(istar, lane);
                wsteps += long_walk_wave<LDS>(istar);
                ++head;
                wave_sync();
                if constexpr (!LDS) {
                    if (__ballot(mine && xv > s0 && xv <= shi)) remark();
                }
                continue;
            }
            int xv[4] = {-1, -1, -1, -1}, xb[4] = {0, 0, 0, 0};
            if (hs != kRewalk) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int j = c * kWave + lane;
                    if (j > kPathLds && j <= K) xv[c] = gpath[hsl * kSamplerPathGlobal + (j - 1 - kPathLds)];
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int j = c * kWave + lane;
                    if (j > kPathLds && j <= K) {
                        xb[c] = (int)((unsigned)xv[c] >> 30);
                        xv[c] &= kVertexMask;
                    }
                }
                if (lane == 0) {
                    xv[0] = s0;
                } else if (lane <= kPathLds) {
                    xv[0] = (int)rob_p[hsl].v[lane - 1];
                    xb[0] = ((int)rob_pb[hsl] >> (2 * (lane - 1))) & 3;
                }
            }
            if (hs == kContinue || hs == kRewalk) {
                // the sequential algorithm for this start against the current tree
                // (all earlier starts are committed).  An overflowed walk whose record misses
                // the tree resumes after its record: the recorded steps become Next pointers.
                const long long k0 = hs == kContinue ? kPath : 0;
                int xs = s0;
                if (hs == kContinue) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (c * kWave + lane <= kPath) htab[c * kWave + lane] = xv[c];
                    wave_sync();
                    if (lane == 0) {
#pragma unroll 10
                        for (int j = 0; j < kPath; ++j) next.set(htab[j], htab[j + 1]);
                    }
                    xs = htab[kPath];
                    wave_sync();
                }
                uint32_t wk0 = (uint32_t)s0;  // the walk's Philox key
                if constexpr (BV) wk0 = (uint32_t)a.skey[s0];
                const long long kk = walk_next<LDS, CT, WT, GL, BV>(bits, next, rp, col, g.hops, lhops, cw, guide, wk0,
                                                                __builtin_amdgcn_readfirstlane(xs), k0, tlo, thi, g.key0,
                                                                g.key1);
                retrace<LDS>(bits, next, nbw, par, bflag, u, s0, htab, stamps, round);
                for (int i = lane; i < 2 * kHashSlots; i += kWave) htab[i] = kWave;
                wsteps += kk;
                wdraws += kk - k0;
                ++head;
                wave_sync();
                if constexpr (!LDS) remark();
                continue;
            }
            // truncation; with the tree state in the records the test's load is ya's chain value too
            int istar = -1, nt = kFree;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (c * kWave <= K && istar < 0) {  // uniform
                    const int j = c * kWave + lane;
                    const bool valid = j >= 1 && j <= K;
                    int nb = kFree;
                    if (valid) {
                        if constexpr (LDS) nb = bits.test(xv[c]) ? 0 : kFree;
                        else nb = bits.nbx(xv[c]);
                    }
                    const uint64_t im = __ballot(nb != kFree);
                    if (im) {
                        istar = c * kWave + __builtin_ctzll(im);
                        nt = __builtin_amdgcn_readlane(nb, __builtin_ctzll(im));
                    }
                }
            }
            if (istar < 0) {
                // an overflowed walk that still misses the tree resumes after its record; for
                // a finished walk this cannot happen, and the re-walk keeps the commit exact
                rob_k[hsl] = (uint8_t)(ended ? kRewalk : kContinue);
                wave_sync();
                continue;
            }
            auto xat = [&](int j) {  // x_j, j uniform
                const int l = j & (kWave - 1);
                const int c = j >> 6;
                int v = __builtin_amdgcn_readlane(xv[0], l);
                if (c == 1) v = __builtin_amdgcn_readlane(xv[1], l);
                if (c == 2) v = __builtin_amdgcn_readlane(xv[2], l);
                if (c == 3) v = __builtin_amdgcn_readlane(xv[3], l);
                return v;
            };
            const int ya = xat(istar);
            int carry;
            if constexpr (LDS) carry = ended && istar == K ? (int)rob_e[hsl].cv : cv_of(ya, load_nbx(nbw, ya));
            else carry = cv_of(ya, nt);
            carry = __builtin_amdgcn_readfirstlane(carry);
            // loop erasure: from b, jump past b's last visit before istar; kept positions per chunk
            uint64_t kept[4] = {0ull, 0ull, 0ull, 0ull};
            if (istar <= kWave) {
                const uint64_t before = istar == kWave ? ~0ull : (1ull << istar) - 1ull;
                int q = 0;
                do {
                    const int b = __builtin_amdgcn_readlane(xv[0], q);
                    const uint64_t mm = __ballot(xv[0] == b) & before;  // holds q
                    q = 63 - __builtin_clzll(mm);
                    kept[0] |= 1ull << q;
                    ++q;
                } while (q < istar);
            } else {
                int q = 0;
                do {
                    const int b = xat(q);
                    int last = q;  // b's last visit: at q or later
#pragma unroll
                    for (int c = 3; c >= 0; --c) {
                        if (last == q && c * kWave < istar) {
                            const uint64_t mm = __ballot(xv[c] == b && c * kWave + lane < istar);
                            if (mm) {
                                const int p = c * kWave + 63 - __builtin_clzll(mm);
                                if (p > last) last = p;
                            }
                        }
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (last >> 6 == c) kept[c] |= 1ull << (last & 63);
                    q = last + 1;
                } while (q < istar);
            }
            // records of the kept positions, attached to ya: x_q's parent is x_{q+1}, its flags the
            // edge bits of step q+1, its nba the next marked kept vertex
            bool inr = false;
#pragma unroll
            for (int c = 3; c >= 0; --c) {
                if (c * kWave < istar) {  // uniform
                    const int hix = c < 3 ? __builtin_amdgcn_readlane(xv[c < 3 ? c + 1 : 3], 0) : 0;
                    const int hib = c < 3 ? __builtin_amdgcn_readlane(xb[c < 3 ? c + 1 : 3], 0) : 0;
                    int nx = __shfl_down(xv[c], 1, kWave), nb = __shfl_down(xb[c], 1, kWave);
                    if (lane == kWave - 1) {
                        nx = hix;
                        nb = hib;
                    }
                    const bool mine = (kept[c] >> lane) & 1ull;
                    const uint64_t m = __ballot(mine && (nb & 2));
                    const uint64_t above = lane < kWave - 1 ? (m & (~0ull << (lane + 1))) : 0ull;
                    const int up = __shfl(xv[c], above ? __builtin_ctzll(above) : 0, kWave);
                    if (mine) {
                        vertex_at(nbw, xv[c]) = (above ? up : carry) | (nb << 30);
                        if (keeps_parent(nb)) vertex_at(par, xv[c]) = nx;
                        bits.set(xv[c]);
                        if constexpr (!LDS) stamps[stamp_slot(xv[c])] = (uint16_t)round;
                        inr = inr || (xv[c] > s0 && xv[c] <= shi);
                    }
                    if (m) carry = __builtin_amdgcn_readlane(xv[c], __builtin_ctzll(m));
                }
            }
            steps += long_walk_lane<LDS>(istar, lane);
            wsteps += long_walk_wave<LDS>(istar);
            ++head;
            wave_sync();
            if constexpr (!LDS) {
                if (__ballot(inr)) remark();
            }
        }
    }

    const long long sum_steps = wsteps + (long long)wave_sum((unsigned long long)steps);
    const long long sum_draws = wdraws + (long long)wave_sum((unsigned long long)draws);
    if (lane == 0) {
        if (a.steps) a.steps[tile] = sum_steps;
        if (a.draws) a.draws[tile] = sum_draws;
    }
    }  // next tile
}

// ======================================================================================
// Records of caller-supplied trees.  The sampler writes each vertex's record as it commits; for
// trees given as parent arrays the same records are built here by pointer jumping, a thread per
// (vertex, tree): 100 trees of R-MAT scale 15 in 0.57 ms a call.  Two words per vertex are doubled
// side by side: anc(v), an ancestor of v (u once reached), whose end tells whether v reaches the
// pivot; and jw(v) = J | done << 31, where J is an ancestor of v such that every vertex
// from parent(v) up to J is unmarked and not u (not done), or J = nba(v) (done).  A round follows
// kJumps pointers, so the covered path grows by a factor of 8; any value that another thread has
// stored keeps the invariants, so threads need no ordering within a round.  A round after one
// that left nothing open returns at once.  A parent array that is not a spanning tree rooted at u
// sets err |= 64 (a vertex on or below a cycle never reaches u).
//
// (One block per tree that built a child list and walked the levels of T took 880 us a launch at
// 21,000 vertices whatever the number of trees: a chain of levels, barriers and hub lists.)
// ======================================================================================
constexpr unsigned kJumpDone = 0x80000000u;
constexpr int kJumps = 7;

__device__ __forceinline__ bool in_tree_ids(int v, int n) { return v >= 0 && v < n; }

// the words of v at the start; *pv = its parent (-1 at u)
__device__ __forceinline__ void jump_start(const IntervalArgs &a, const int *__restrict__ par, int v, int *anc,
                                           unsigned *jw, int *pv) {
    const int n = a.n, u = a.u;
    *anc = u;
    *jw = (unsigned)u | kJumpDone;
    *pv = -1;
    if (v == u) return;
    const int p = par[v];
    *pv = p;
    if (!in_tree_ids(p, n) || p == v) {
        atomicOr(a.err, 64);
    } else if (p != u) {
        const int pp = par[p];
        const bool marked = in_tree_ids(pp, n) && (mark_bits(p, a.bflag[p], pp, a.bflag[pp]) & kMarkBit);
        *anc = p;
        *jw = (unsigned)p | (marked ? kJumpDone : 0u);
    }
}

// a round of v on the words in memory; true if one of its words is still open
template <typename W>
__device__ __forceinline__ bool jump_round(int u, int v, int *anc, W *jw) {
    bool more = false;
    int x = anc[v];
    if (x != u) {
        for (int i = 0; i < kJumps && x != u; ++i) x = anc[x];
        anc[v] = x;
        more = x != u;
    }
    unsigned w = (unsigned)jw[v];
    if (!(w & kJumpDone)) {
        for (int i = 0; i < kJumps && !(w & kJumpDone); ++i) w = (unsigned)jw[w];
        jw[v] = (W)w;
        more = more || !(w & kJumpDone);
    }
    return more;
}

// the word nba | flags of v once the rounds are over
__device__ __forceinline__ int jump_word(const IntervalArgs &a, int v, int anc, unsigned w, int pv) {
    if (v == a.u) return v;
    if (anc != a.u) atomicOr(a.err, 64);
    const int nba = (w & kJumpDone) ? (int)(w & ~kJumpDone) : a.u;  // not done: on or below a cycle
    return nba | (in_tree_ids(pv, a.n) ? mark_bits(v, a.bflag[v], pv, a.bflag[pv]) : 0);
}

// open[0] = 1, open[1 .. kTreeJumpRounds] = 0 for the rounds
__global__ __launch_bounds__(256) void tree_jump_init_kernel(IntervalArgs a, int *__restrict__ open) {
    const int v = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.y == 0 && v <= kTreeJumpRounds) open[v] = v == 0;
    if (v >= a.n) return;
    int anc, pv;
    unsigned jw;
    jump_start(a, a.par + (long long)blockIdx.y * a.par_stride, v, &anc, &jw, &pv);
    a.scratch[(long long)blockIdx.y * a.scratch_stride + v] = anc;
    int *rec = a.rec + (long long)blockIdx.y * 2 * a.rec_stride;
    rec[v] = (int)jw;
    rec[a.rec_stride + v] = pv;
}

// one round; open[0]: the round before left something open, open[1]: this one did
__global__ __launch_bounds__(256) void tree_jump_kernel(IntervalArgs a, int *__restrict__ open) {
    if (open[0] == 0) return;  // uniform over the grid
    const int v = blockIdx.x * 256 + threadIdx.x;
    bool more = false;
    if (v < a.n)
        more = jump_round(a.u, v, a.scratch + (long long)blockIdx.y * a.scratch_stride,
                          a.rec + (long long)blockIdx.y * 2 * a.rec_stride);
    if (__any(more) && lane_id() == 0) open[1] = 1;
}

__global__ __launch_bounds__(256) void tree_records_kernel(IntervalArgs a) {
    const int v = blockIdx.x * 256 + threadIdx.x;
    if (v >= a.n) return;
    int *rec = a.rec + (long long)blockIdx.y * 2 * a.rec_stride;
    rec[v] = jump_word(a, v, a.scratch[(long long)blockIdx.y * a.scratch_stride + v], (unsigned)rec[v],
                       rec[a.rec_stride + v]);
}

// A small graph: the same rounds in one launch, a block per tree, the words in LDS.  Below a
// thousand vertices the launches were most of the call (path of two vertices, 8 trees two at a time:
// 0.345 ms a call, 0.239 before the rounds had a launch each, now 0.129).
constexpr int kTreeSmallMaxN = 1024;

__global__ __launch_bounds__(256) void tree_records_small_kernel(IntervalArgs a, int rounds) {
    __shared__ int anc[kTreeSmallMaxN], pv[kTreeSmallMaxN];
    __shared__ unsigned jw[kTreeSmallMaxN];
    const int *__restrict__ par = a.par + (long long)blockIdx.x * a.par_stride;
    for (int v = threadIdx.x; v < a.n; v += 256) jump_start(a, par, v, &anc[v], &jw[v], &pv[v]);
    for (int r = 0; r < rounds; ++r) {
        __syncthreads();
        for (int v = threadIdx.x; v < a.n; v += 256) jump_round(a.u, v, anc, jw);
    }
    __syncthreads();
    int *rec = a.rec + (long long)blockIdx.x * 2 * a.rec_stride;
    for (int v = threadIdx.x; v < a.n; v += 256) {
        rec[v] = jump_word(a, v, anc[v], jw[v], pv[v]);
        rec[a.rec_stride + v] = pv[v];
    }
}

// ======================================================================================
// Aggregation (Algorithm 2), on the records: for v != u,
//   c_T(v) = [parent_T(v) = parB(v)]
//          + sum over marked strict T-ancestors x of v lying on P(v) of
//              +1 if parent_T(x) = parB(x),  -1 if parB(parent_T(x)) = x and parent_T(x) on P(v),
// which equals Algorithm 2's signed count term by term.  Thread per vertex over a chunk of
// resident trees; one int64 atomic per vertex and chunk, skipped when the sum is zero.  A chain
// step reads the word nba(x) | flags alone; parent_T(x) only for a backward x on P(v).
//
// "On P(v)", two forms.  PL > 0 (shallow B_u): P(v) has at most ecc(u) - 1 <= PL vertices p_1 ..
// beside v and u, which the thread keeps in registers, p_0 = v: x is on P(v) if it is one of
// them, and a backward x = p_i counts if parent_T(x) = p_{i-1}, its B_u child towards v.  PL = 0:
// the B_u subtree test pre_B(x) <= pre_B(v) < pre_B(x) + size_B(x).  What bounds the kernel is
// its gathers, one per lane and chain vertex for the word and, with PL = 0, one more for the
// interval, and the instructions around them: with the records as pairs {parent, word}, 24 vector
// instructions a chain step, half of the vector issue rate at R-MAT scale 22.
// ======================================================================================
// WT: weighted graph, the edge (parB(b), b) of P(v) counts +-F[b] (Ohm's-law factor in fixed
// point) instead of +-1.
template <bool WT, int CH, int PL>
__global__ __launch_bounds__(256) void aggregate_kernel(AggregateArgs a) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= a.n || v == a.u) return;
    const int t0 = blockIdx.y * CH;
    const int nt = min(a.ntrees - t0, CH);
    const unsigned u = (unsigned)a.u;
    const int2 *__restrict__ bint = a.bint;
    const int *__restrict__ parB = a.parB;
    const int pv = PL ? 0 : bint[v].x;
    const int *__restrict__ rec0 = a.rec + (long long)t0 * 2 * a.rec_stride;  // uniform
    // word and parent of x in tree i: a uniform base and a 32-bit offset (4 x < 2^32)
    auto word = [&](int i, unsigned x) {
        return *reinterpret_cast<const int *>(reinterpret_cast<const char *>(rec0 + (long long)i * 2 * a.rec_stride) +
                                              (x << 2));
    };
    auto parent = [&](int i, unsigned x) {
        return *reinterpret_cast<const int *>(
            reinterpret_cast<const char *>(rec0 + (long long)(2 * i + 1) * a.rec_stride) + (x << 2));
    };
    // The chains of the chunk's trees are walked in lockstep, one step of every unfinished
    // chain per round, so their independent loads are in flight together.
    using Acc = typename std::conditional<WT, long long, int>::type;
    const long long *__restrict__ F = a.F;
    const Acc fv = WT ? (Acc)F[v] : (Acc)1;
    unsigned x[CH];
    Acc sum = 0;
    {
        int w[CH];
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            w[i] = (int)u;  // no such tree: nothing to add, no chain
            if (i < nt) w[i] = word(i, (unsigned)v);
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if constexpr (WT) sum += (w[i] & kFwdBit) ? fv : (Acc)0;
            else sum += (w[i] >> 30) & 1;
            x[i] = (unsigned)nba_of(w[i]);
        }
    }
    int p[PL + 1];  // p_0 = v, p_1 = parB(v), ..; -1 from u on
    p[0] = v;
    if constexpr (PL > 0) {
        int b = parB[v];
#pragma unroll
        for (int i = 1; i <= PL; ++i) {
            p[i] = b != a.u ? b : -1;
            if (i < PL && b != a.u) b = parB[b];
        }
    }
    // a chain visits each T-ancestor at most once: n rounds bound it
    for (int round = 0; round < a.n; ++round) {
        int w[CH];
        int2 bx[CH];
        bool act = false;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (x[i] != u) {
                act = true;
                w[i] = word(i, x[i]);
                if constexpr (PL == 0) bx[i] = bint[x[i]];
            }
        }
        if (!act) break;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (x[i] != u) {
                // a forward x counts +1 if x is on P(v); a backward x counts -1 if parent_T(x),
                // a B_u child of x, is on P(v), which needs x on P(v) first
                bool on;
                if constexpr (PL > 0) {
                    on = (int)x[i] == p[1];
#pragma unroll
                    for (int j = 2; j <= PL; ++j) on |= (int)x[i] == p[j];
                } else {
                    on = bx[i].x <= pv && pv < bx[i].x + bx[i].y;
                }
                if (on) {
                    if (w[i] & kFwdBit) {
                        if constexpr (WT) sum += F[x[i]];
                        else ++sum;
                    } else {
                        const int q = parent(i, x[i]);
                        bool below = false;
                        if constexpr (PL > 0) {
#pragma unroll
                            for (int j = 1; j <= PL; ++j) below |= (int)x[i] == p[j] && q == p[j - 1];
                        } else {
                            const int2 bp = bint[q];
                            below = bp.x <= pv && pv < bp.x + bp.y;
                        }
                        if (below) {
                            if constexpr (WT) sum -= F[q];
                            else --sum;
                        }
                    }
                }
                x[i] = (unsigned)nba_of(w[i]);
            }
        }
    }
    if (sum != 0) atomicAdd((unsigned long long *)&a.counts[v], (unsigned long long)(long long)sum);
}

// Subtree intervals of B_u, level by level over the whole grid (B_u has ecc(u) + 1 levels):
// sizes bottom-up (each vertex adds its finished size to its parent), then pre-order
// numbers top-down (each vertex takes the next free range under its parent; the order of
// siblings is whatever the atomics give, and any order is a valid nesting).
__global__ void bsub_init_kernel(int n, int u, int *__restrict__ sz, int *__restrict__ cur, int *__restrict__ pre) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    sz[v] = 1;
    if (v == u) {
        pre[v] = 0;
        cur[v] = 1;
    }
}
// Children of one hub make up most of a level in small-world graphs; the lanes of a wave
// that share the parent of the wave's first active lane combine into one atomic.
__global__ __launch_bounds__(256) void bsub_size_kernel(int n, int d, const int *__restrict__ dist,
                                                        const int *__restrict__ parB, int *__restrict__ sz) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    const bool act = v < n && dist[v] == d;
    const int p = act ? parB[v] : -1, val = act ? sz[v] : 0;
    const uint64_t am = __ballot(act);
    if (!am) return;
    const int leader = __builtin_ctzll(am);
    const int lp = __shfl(p, leader, kWave);
    const bool same = act && p == lp;
    const int tot = wave_sum(same ? val : 0);
    if (lane_id() == leader) atomicAdd(&sz[lp], tot);
    if (act && !same) atomicAdd(&sz[p], val);
}
__global__ __launch_bounds__(256) void bsub_pre_kernel(int n, int d, const int *__restrict__ dist,
                                                       const int *__restrict__ parB, const int *__restrict__ sz,
                                                       int *__restrict__ cur, int *__restrict__ pre) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    const bool act = v < n && dist[v] == d;
    const int p = act ? parB[v] : -1, val = act ? sz[v] : 0;
    const uint64_t am = __ballot(act);
    if (!am) return;
    const int leader = __builtin_ctzll(am);
    const int lp = __shfl(p, leader, kWave);
    const bool same = act && p == lp;
    const int incl = wave_incl_scan(same ? val : 0);
    const int tot = __shfl(incl, kWave - 1, kWave);
    int base = 0;
    if (lane_id() == leader) base = atomicAdd(&cur[lp], tot);
    base = __shfl(base, leader, kWave);
    int pv = 0;
    if (same) pv = base + incl - val;
    else if (act) pv = atomicAdd(&cur[p], val);
    if (act) {
        pre[v] = pv;
        cur[v] = pv + 1;
    }
}
__global__ void bsub_pack_kernel(int n, const int *__restrict__ parB, const int *__restrict__ pre,
                                 const int *__restrict__ sz, int2 *__restrict__ bint, int *__restrict__ bflag) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const int pb = parB[v], z = sz[v];
    bint[v] = make_int2(pre[v], z);
    bflag[v] = (int)((unsigned)(pb + 1) | (z > 1 ? 0x80000000u : 0u));
}

// The pivot by BFS sweeps for a small graph, in one workgroup and with no host round trip:
// the same first source (largest degree, then smallest ID), the same level-synchronous BFS, the
// same bounds (the distances of the first sweep, then their running maximum) and next source
// (the farthest vertex, then smallest ID) as sweep_update_kernel, and the same choice (smallest
// bound, then smallest ID) as argmin_bound_kernel.  *pivot receives the choice.
constexpr int kSweepThreads = 1024;

__device__ __forceinline__ unsigned long long block_max_key(unsigned long long key, unsigned long long *sh) {
#pragma unroll
    for (int dd = 32; dd > 0; dd >>= 1) {
        const unsigned long long o = __shfl_xor(key, dd, 64);
        key = o > key ? o : key;
    }
    if ((threadIdx.x & (kWave - 1)) == 0) sh[threadIdx.x / kWave] = key;
    __syncthreads();
    unsigned long long r = 0;
    for (int i = 0; i < kSweepThreads / kWave; ++i) r = sh[i] > r ? sh[i] : r;
    __syncthreads();  // every thread has read sh before it is written again
    return r;
}

template <int G>
__global__ __launch_bounds__(kSweepThreads) void sweep_small_kernel(RowMap m, int sweeps, int *__restrict__ dist,
                                                                    int *__restrict__ bound, int *__restrict__ pivot) {
    __shared__ unsigned long long shk[kSweepThreads / kWave];
    __shared__ int found;
    const int n = m.n, tid = threadIdx.x;
    const int nh = *m.nheavy;
    unsigned long long key = 0;
    for (int v = tid; v < n; v += kSweepThreads) {
        const unsigned long long k = ((unsigned long long)(unsigned)(m.rp[v + 1] - m.rp[v]) << 32) |
                                     (unsigned long long)(0xFFFFFFFFu - (unsigned)v);
        key = k > key ? k : key;
    }
    int src = (int)(0xFFFFFFFFu - (unsigned)(block_max_key(key, shk) & 0xFFFFFFFFull));
    for (int it = 0; it < sweeps; ++it) {
        for (int v = tid; v < n; v += kSweepThreads) dist[v] = (v == src) ? 0 : INT_MAX;
        for (int d = 0;; ++d) {
            if (tid == 0) found = 0;
            __syncthreads();
            int any = 0;
            for (int h = 0; h < nh; ++h) {
                const int v = m.heavy[h];
                if (dist[v] != d) continue;  // uniform in the block
                for (int e = m.rp[v] + tid; e < m.rp[v + 1]; e += kSweepThreads) {
                    const int y = m.col[e];
                    if (dist[y] > d + 1) {
                        dist[y] = d + 1;
                        any = 1;
                    }
                }
            }
            constexpr int rows_per_tile = kSweepThreads / G;
            const int g = tid / G, l = tid % G;
            for (int base = 0; base < n; base += rows_per_tile) {
                const int v = base + g;
                if (v >= n || dist[v] != d) continue;
                const int lo = m.rp[v], hi = m.rp[v + 1];
                if (hi - lo > m.heavy_thresh) continue;
                for (int e = lo + l; e < hi; e += G) {
                    const int y = m.col[e];
                    if (dist[y] > d + 1) {
                        dist[y] = d + 1;
                        any = 1;
                    }
                }
            }
            if (any) found = 1;
            __syncthreads();
            const int f = found;
            __syncthreads();  // every thread has read `found` before it is reset
            if (!f) break;
        }
        key = 0;
        for (int v = tid; v < n; v += kSweepThreads) {
            const int d = dist[v];
            bound[v] = it == 0 ? d : max(bound[v], d);
            const unsigned long long k = ((unsigned long long)(unsigned)d << 32) |
                                         (unsigned long long)(0xFFFFFFFFu - (unsigned)v);
            key = k > key ? k : key;
        }
        src = (int)(0xFFFFFFFFu - (unsigned)(block_max_key(key, shk) & 0xFFFFFFFFull));
    }
    key = 0;
    for (int v = tid; v < n; v += kSweepThreads) {
        const unsigned long long k = ((unsigned long long)(0x7FFFFFFFu - (unsigned)bound[v]) << 32) |
                                     (unsigned long long)(0xFFFFFFFFu - (unsigned)v);
        key = k > key ? k : key;
    }
    key = block_max_key(key, shk);
    if (tid == 0) *pivot = (int)(0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull));
}

// Set-up of a small graph in one workgroup: the BFS levels (the same minimum-ID parent
// rule as bfs_level_kernel), the connectivity check, and the subtree intervals and flag
// words of B_u (as the bsub_* kernels).  out[0] = ecc(u), out[1] = 1 if a vertex is
// unreached.  scratch holds 3n ints.
constexpr int kSetupThreads = 1024;

template <int G>
__global__ __launch_bounds__(kSetupThreads) void setup_small_kernel(RowMap m, int u, int *__restrict__ dist,
                                                                    int *__restrict__ parB, int *__restrict__ scratch,
                                                                    int2 *__restrict__ bint, int *__restrict__ bflag,
                                                                    int *__restrict__ out) {
    __shared__ int found, unreached;
    const int n = m.n, tid = threadIdx.x;
    int *__restrict__ sz = scratch;
    int *__restrict__ cur = scratch + n;
    int *__restrict__ pre = scratch + 2 * n;
    for (int v = tid; v < n; v += kSetupThreads) {
        dist[v] = (v == u) ? 0 : INT_MAX;
        parB[v] = (v == u) ? -1 : INT_MAX;
        sz[v] = 1;
    }
    if (tid == 0) unreached = 0;
    const int nh = *m.nheavy;
    int d = 0;
    for (;; ++d) {
        if (tid == 0) found = 0;
        __syncthreads();
        int any = 0;
        for (int h = 0; h < nh; ++h) {
            const int v = m.heavy[h];
            if (dist[v] != d) continue;  // uniform in the block
            for (int e = m.rp[v] + tid; e < m.rp[v + 1]; e += kSetupThreads) {
                const int y = m.col[e];
                const int dy = dist[y];
                if (dy > d) {
                    atomicMin(&parB[y], v);
                    if (dy != d + 1) dist[y] = d + 1;
                    any = 1;
                }
            }
        }
        constexpr int rows_per_tile = kSetupThreads / G;
        const int g = tid / G, l = tid % G;
        for (int base = 0; base < n; base += rows_per_tile) {
            const int v = base + g;
            if (v >= n || dist[v] != d) continue;
            const int lo = m.rp[v], hi = m.rp[v + 1];
            if (hi - lo > m.heavy_thresh) continue;
            for (int e = lo + l; e < hi; e += G) {
                const int y = m.col[e];
                const int dy = dist[y];
                if (dy > d) {
                    atomicMin(&parB[y], v);
                    if (dy != d + 1) dist[y] = d + 1;
                    any = 1;
                }
            }
        }
        if (any) found = 1;
        __syncthreads();
        const int f = found;
        __syncthreads();  // every thread has read `found` before it is reset
        if (!f) break;
    }
    const int ecc = d;
    for (int v = tid; v < n; v += kSetupThreads)
        if (dist[v] == INT_MAX) unreached = 1;
    __syncthreads();
    if (unreached) {
        if (tid == 0) {
            out[0] = ecc;
            out[1] = 1;
        }
        return;
    }
    // subtree sizes bottom-up, then pre-order ranges top-down, level by level
    for (int dd = ecc; dd >= 1; --dd) {
        for (int v = tid; v < n; v += kSetupThreads)
            if (dist[v] == dd) atomicAdd(&sz[parB[v]], sz[v]);
        __syncthreads();
    }
    if (tid == 0) {
        pre[u] = 0;
        cur[u] = 1;
    }
    __syncthreads();
    for (int dd = 1; dd <= ecc; ++dd) {
        for (int v = tid; v < n; v += kSetupThreads) {
            if (dist[v] == dd) {
                const int pv = atomicAdd(&cur[parB[v]], sz[v]);
                pre[v] = pv;
                cur[v] = pv + 1;
            }
        }
        __syncthreads();
    }
    for (int v = tid; v < n; v += kSetupThreads) {
        const int pb = parB[v], z = sz[v];
        bint[v] = make_int2(pre[v], z);
        bflag[v] = (int)((unsigned)(pb + 1) | (z > 1 ? 0x80000000u : 0u));
    }
    if (tid == 0) {
        out[0] = ecc;
        out[1] = 0;
    }
}


// parents[i][v] = rec_i[v].parent
__global__ void extract_parents_kernel(int n, int ntrees, const int *__restrict__ rec, long long rec_stride,
                                       int *__restrict__ out) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)n * ntrees) return;
    const long long t = i / n, v = i - t * n;
    out[i] = rec[(2 * t + 1) * rec_stride + v];
}

// ======================================================================================
// Measures that depend only on diag(L^+) (section on electrical closeness, Eq. elec-farness;
// Lemma on normalized random-walk betweenness; Kirchhoff index appendix):
//   tr = sum_v diag[v], farness[v] = n diag[v] + tr, closeness[v] = (n-1) / farness[v],
//   nrwb[v] = 1/n + tr / ((n-1) farness[v]), Kirchhoff index = n tr.
// The trace is summed in an order that depends on n alone (deterministic).
// ======================================================================================
constexpr int kTraceThreads = 1024;
// Beyond kTraceOneMax entries one workgroup's loads in flight bound the sum (n = 2.4M: 592 us, 33
// GB/s); blocks of kTracePerBlock entries each, whose partial sums a last workgroup adds, read it
// at memory speed (all measures of n = 2.4M: 587 us before, 42 us).  The call has no workspace, so
// the partial sums go to the front of an output array (overwritten by the measures afterwards)
// that does not overlap the diagonal; a call without such an array keeps the one workgroup.
constexpr long long kTraceOneMax = 16384, kTracePerBlock = 4096;

__global__ __launch_bounds__(kTraceThreads) void trace_kernel(long long n, const double *__restrict__ diag,
                                                              double *__restrict__ scalars) {
    __shared__ double sh[kTraceThreads / kWave];
    double acc = 0.0;
    for (long long v = threadIdx.x; v < n; v += kTraceThreads) acc += diag[v];
    acc = block_sum_t<double>(acc, sh);
    if (threadIdx.x == 0) {
        scalars[0] = acc;
        scalars[1] = (double)n * acc;
    }
}

__global__ __launch_bounds__(256) void trace_partial_kernel(long long n, const double *__restrict__ diag,
                                                            double *__restrict__ part) {
    __shared__ double sh[256 / kWave];
    const long long base = (long long)blockIdx.x * kTracePerBlock + threadIdx.x;
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < kTracePerBlock / 256; ++j) {
        const long long v = base + j * 256;
        acc += v < n ? diag[v] : 0.0;
    }
    acc = block_sum_t<double>(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

__global__ __launch_bounds__(kTraceThreads) void trace_finish_kernel(long long n, int nparts,
                                                                     const double *__restrict__ part,
                                                                     double *__restrict__ scalars) {
    __shared__ double sh[kTraceThreads / kWave];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nparts; i += kTraceThreads) acc += part[i];
    acc = block_sum_t<double>(acc, sh);
    if (threadIdx.x == 0) {
        scalars[0] = acc;
        scalars[1] = (double)n * acc;
    }
}

__global__ __launch_bounds__(256) void centrality_kernel(long long n, const double *__restrict__ diag,
                                                         const double *__restrict__ scalars,
                                                         double *__restrict__ farness, double *__restrict__ closeness,
                                                         double *__restrict__ nrwb) {
    const long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const double tr = scalars[0];
    const double f = (double)n * diag[v] + tr;
    if (farness) farness[v] = f;
    if (closeness) closeness[v] = (double)(n - 1) / f;
    if (nrwb) nrwb[v] = 1.0 / (double)n + tr / ((double)(n - 1) * f);
}

// ======================================================================================
// Spanning-edge counts (Kirchhoff index appendix: for each edge, the number of sampled
// USTs it appears in).  Thread per vertex v != u over a chunk of resident trees: the edge
// v -> parent_T(v) is found by binary search in v's own ascending row (short for the
// children of hubs) and counted at that position; equal positions in a row of trees add
// with one atomic.  edge_fold_kernel then moves every count at an entry (a, b), a > b, to
// the entry (b, a), so each undirected edge is counted at (min, max).
// ======================================================================================
__global__ __launch_bounds__(256) void edge_count_kernel(EdgeCountArgs a) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= a.n || v == a.u) return;
    const int t0 = blockIdx.y * a.trees_per_chunk;
    const int t1 = min(a.ntrees, t0 + a.trees_per_chunk);
    long long cur = -1;
    int c = 0;
    for (int t = t0; t < t1; ++t) {
        const int p = a.rec[(2ll * t + 1) * a.rec_stride + v];
        const int end = a.rp[v + 1], lo = row_lower_bound(a.col, a.rp[v], end, p);
        if (lo == end || a.col[lo] != p) continue;  // not a neighbour: never for a sampled tree
        if (lo == cur) {
            ++c;
        } else {
            if (c) atomicAdd((unsigned long long *)&a.counts[cur], (unsigned long long)c);
            cur = lo;
            c = 1;
        }
    }
    if (c) atomicAdd((unsigned long long *)&a.counts[cur], (unsigned long long)c);
}

// Thread per entry e = (a, b) with a > b and a nonzero count: add it to the entry (b, a)
// (binary search in row b) and clear it.  Entries (b, a) with b < a are never cleared, so
// each receives from exactly one entry.  The row a of entry e comes from a binary search
// over the row pointers.
__global__ __launch_bounds__(256) void edge_fold_kernel(int n, long long nnz, const int *__restrict__ rp,
                                                        const int *__restrict__ col, long long *__restrict__ counts) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    const long long c = counts[e];
    if (c == 0) return;
    int lo = 0, hi = n;  // largest a with rp[a] <= e
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (rp[mid] <= e) lo = mid;
        else hi = mid;
    }
    const int a = lo, b = col[e];
    if (b >= a) return;
    const int end = rp[b + 1], l = row_lower_bound(col, rp[b], end, a);
    if (l == end || col[l] != a) return;  // asymmetric input: left where it is
    atomicAdd((unsigned long long *)&counts[l], (unsigned long long)c);
    counts[e] = 0;
}

// Edge measures from spanning-edge counts (Kirchhoff index appendix): thread per CSR entry
// e = (a, b); the count sits at the entry (min, max) of the edge (the mirror entry (b, a) is
// found by binary search in row b); lev = c / q, r = lev / w(e), denom = 1 - (1 - theta) lev.
__global__ __launch_bounds__(256) void edge_resistance_kernel(int n, long long nnz, const long long *__restrict__ rp,
                                                              const int *__restrict__ col,
                                                              const double *__restrict__ w,
                                                              const long long *__restrict__ counts, double q,
                                                              double theta, double *__restrict__ r,
                                                              double *__restrict__ denom) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    int lo = 0, hi = n;  // the row a: the largest a with rp[a] <= e
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (rp[mid] <= e) lo = mid;
        else hi = mid;
    }
    const int a = lo, b = col[e];
    long long c = counts[e];
    if (b < a) {  // the count is at the mirror entry (b, a)
        long long l = rp[b], h = rp[b + 1];
        c = 0;
        while (l < h) {
            const long long mid = (l + h) >> 1;
            const int cm = col[mid];
            if (cm == a) {
                c = counts[mid];
                break;
            }
            if (cm < a) l = mid + 1;
            else h = mid;
        }
    }
    {
        // each operation rounded on its own, as the definition reads: no contraction into a fused
        // multiply-add
#pragma clang fp contract(off)
        const double lev = (double)c / q;
        if (r) r[e] = lev / (w ? w[e] : 1.0);
        if (denom) denom[e] = 1.0 - (1.0 - theta) * lev;
    }
}

// Final fill (Algorithm 1; Eq. diag-comp): diag[u] = x[u], diag[v] = R[v]/tau - x[u] + 2 x[v]
// ======================================================================================
// Weighted graphs (Section "Generalizations").  Set-up only: the running conductance sums
// of every row (the sampler's step table and the Laplacian's diagonal), the weight checks,
// the B-path resistances and the fixed-point edge factors of Algorithm 2.
// ======================================================================================
// Running sums taken left to right, so every device (and the CPU oracle) gets the same FP64
// sums: cw[e] = w[row start] + ... + w[e], wdeg[v] = the row total.  One thread per light
// row; rows above `heavy_thresh` entries are left to row_cumsum_heavy_kernel.
__global__ __launch_bounds__(256) void row_cumsum_kernel(int n, const int *__restrict__ rp, const double *__restrict__ w,
                                                         int heavy_thresh, double *__restrict__ cw,
                                                         double *__restrict__ wdeg) {
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        const int lo = rp[v], end = rp[v + 1];
        if (end - lo > heavy_thresh) continue;
        wdeg[v] = row_running_sums(w, cw, lo, end);
    }
}

// A heavy row per wavefront: each 64-entry chunk is loaded at once (the next one while the
// current is summed), and the running sum passes through the lanes in order, one addition
// per entry as in the sequential loop; lane k keeps the sum up to its own entry.
__global__ __launch_bounds__(64) void row_cumsum_heavy_kernel(const int *__restrict__ rp, const double *__restrict__ w,
                                                              const int *__restrict__ heavy, const int *__restrict__ nheavy,
                                                              double *__restrict__ cw, double *__restrict__ wdeg) {
    const int nh = *nheavy;
    const int lane = threadIdx.x;
    for (int h = blockIdx.x; h < nh; h += gridDim.x) {
        const int v = heavy[h];
        const int r0 = rp[v], end = rp[v + 1];
        double run = 0.0;
        const uint32_t rend = (uint32_t)end;
        auto chunk = [&](uint32_t base) { return base + lane < rend ? w[base + lane] : 0.0; };
        double wn = chunk((uint32_t)r0);
        row_each(r0, end, 0, kWave, [&](uint32_t base) {
            const double wc = wn;
            wn = chunk(base + kWave);
            const int cnt = (int)min((uint32_t)kWave, rend - base);
            const long long bits = __double_as_longlong(wc);
            const int lo = (int)(bits & 0xFFFFFFFFll), hi = (int)(bits >> 32);
            double mine = 0.0;
            for (int k = 0; k < cnt; ++k) {
                const long long bk = ((long long)(unsigned)__builtin_amdgcn_readlane(hi, k) << 32) |
                                     (long long)(unsigned)__builtin_amdgcn_readlane(lo, k);
                run += __longlong_as_double(bk);
                if (lane == k) mine = run;
            }
            if (lane < cnt) cw[base + lane] = mine;
        });
        if (lane == 0) wdeg[v] = run;
    }
}

// Guide of the weighted step search, one thread per CSR entry e = (row v, bucket i):
// guide[e] = the first j (at most deg-1) with C[j] > t(w_i), w_i = ceil(i 2^32 / deg) the
// smallest word of bucket i.  The row is found by a binary search over the row pointers.
__global__ __launch_bounds__(256) void step_guide_kernel(int n, int nnz, const int *__restrict__ rp,
                                                         const double *__restrict__ cw, int *__restrict__ guide) {
    row_each(0, nnz, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x, [&](uint32_t slot) {
        const int e = (int)slot;
        int lo = 0, hi = n - 1;  // the last v with rp[v] <= e
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (rp[mid] <= e) lo = mid;
            else hi = mid - 1;
        }
        const int r0 = rp[lo], deg = rp[lo + 1] - r0, i = e - r0;
        const unsigned long long wi = (((unsigned long long)i << 32) + (unsigned long long)(deg - 1)) / (unsigned)deg;
        const double ti = ((double)wi * 0x1p-32) * cw[r0 + deg - 1];
        int a = 0, b = deg - 1;  // the first j with ti < C[j], or deg-1
        while (a < b) {
            const int mid = (a + b) >> 1;
            if (ti < cw[r0 + mid]) b = mid;
            else a = mid + 1;
        }
        guide[e] = a;
    });
}

// err |= 64 if a conductance is not positive and finite or differs from its mirror entry
__global__ __launch_bounds__(256) void check_weights_kernel(int n, const int *__restrict__ rp, const int *__restrict__ col,
                                                            const double *__restrict__ w, int *__restrict__ err) {
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
        bool bad = false;
        for (int e = rp[v]; e < rp[v + 1]; ++e) {
            const double we = w[e];
            const int x = col[e];
            if (!(we > 0.0) || !isfinite(we) || x < 0 || x >= n) { bad = true; break; }
            const int f = find_in_row(col, rp[x], rp[x + 1], v);
            if (f < 0 || w[f] != we) { bad = true; break; }
        }
        if (bad) atomicOr(err, 64);
    }
}

// wB[v] = w(v, parB(v)) (0 at u), then rho(v) = sum of 1 / wB over P(v) from v towards u;
// the largest rho into *rmax_bits (bits of a non-negative double order like the values)
__global__ __launch_bounds__(256) void b_edge_weight_kernel(int n, int u, const int *__restrict__ rp,
                                                            const int *__restrict__ col, const double *__restrict__ w,
                                                            const int *__restrict__ parB, double *__restrict__ wB) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    double wb = 0.0;
    if (v != u) {
        const int f = find_in_row(col, rp[v], rp[v + 1], parB[v]);
        wb = f >= 0 ? w[f] : 0.0;  // parB(v) is a neighbour of v
    }
    wB[v] = wb;
}
__global__ __launch_bounds__(256) void bpath_resist_kernel(int n, int u, const int *__restrict__ parB,
                                                           const double *__restrict__ wB,
                                                           unsigned long long *__restrict__ rmax_bits) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    double r = 0.0;
    if (v < n)
        for (int b = v; b != u; b = parB[b]) r += 1.0 / wB[b];
    unsigned long long bits = (unsigned long long)__double_as_longlong(r);
    for (int d = kWave / 2; d > 0; d >>= 1) bits = max(bits, (unsigned long long)__shfl_xor((long long)bits, d, kWave));
    if (lane_id() == 0 && bits) atomicMax(rmax_bits, bits);
}

// F[v] = llround(2^shift / wB[v]), F[u] = 0
__global__ void fixed_weights_kernel(int n, int u, const double *__restrict__ wB, double scale, long long *__restrict__ F) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    F[v] = v == u ? 0ll : llround(scale / wB[v]);
}

// walk steps and draws of `cnt` trees added to totals[0], totals[1] (one block)
__global__ __launch_bounds__(256) void sum_walks_kernel(int cnt, const long long *__restrict__ steps,
                                                        const long long *__restrict__ draws,
                                                        unsigned long long *__restrict__ totals) {
    long long a = 0, b = 0;
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
        a += steps[i];
        b += draws[i];
    }
    for (int d = kWave / 2; d > 0; d >>= 1) {
        a += __shfl_xor(a, d, kWave);
        b += __shfl_xor(b, d, kWave);
    }
    if (lane_id() == 0) {
        atomicAdd(&totals[0], (unsigned long long)a);
        atomicAdd(&totals[1], (unsigned long long)b);
    }
}

// walk steps and draws of a batch's tiles added to their member's totals (totals[2 g], totals[2 g + 1])
__global__ __launch_bounds__(256) void tile_walks_kernel(int cnt, const WilsonTile *__restrict__ tiles,
                                                         const long long *__restrict__ steps,
                                                         const long long *__restrict__ draws,
                                                         unsigned long long *__restrict__ totals) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cnt) return;
    const int g = tiles[i].graph;
    atomicAdd(&totals[2 * g], (unsigned long long)steps[i]);
    atomicAdd(&totals[2 * g + 1], (unsigned long long)draws[i]);
}

// den = tau, or tau 2^k for the fixed-point counts of a weighted graph
__global__ void combine_kernel(int n, int u, double den, const long long *__restrict__ counts,
                               const double *__restrict__ x, double *__restrict__ diag) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    const double xu = x[u];
    diag[v] = (v == u) ? xu : (double)counts[v] / den - xu + 2.0 * x[v];
}

__global__ void philox_words_kernel(uint32_t key0, uint32_t key1, long long t, int s, long long k0, long long count,
                                    uint32_t *__restrict__ out) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const long long k = k0 + i;
    const uint4 o = philox4x32_10(make_uint4((uint32_t)(k >> 2), (uint32_t)s, (uint32_t)(unsigned long long)t,
                                             (uint32_t)((unsigned long long)t >> 32)), key0, key1);
    const int q = (int)(k & 3);
    out[i] = q == 0 ? o.x : (q == 1 ? o.y : (q == 2 ? o.z : o.w));
}

// ======================================================================================
// launchers
// ======================================================================================
static inline int blocks_for(long long n, int bs) { return (int)((n + bs - 1) / bs); }

hipError_t launch_col_to_u16(long long nnz, const int *col, unsigned short *col16, hipStream_t st) {
    col_to_u16_kernel<<<blocks_for(nnz, 256), 256, 0, st>>>(nnz, col, col16);
    return hipGetLastError();
}
hipError_t launch_rp_to_i32(int n, const long long *rp64, int *rp32, hipStream_t st) {
    rp_to_i32_kernel<<<blocks_for(n + 1, 256), 256, 0, st>>>(n, rp64, rp32);
    return hipGetLastError();
}
hipError_t launch_validate(int n, long long nnz, const long long *rp64, const int *col, int *err, hipStream_t st) {
    validate_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, nnz, rp64, col, err);
    return hipGetLastError();
}
hipError_t launch_argmax_degree(int n, const int *rp, unsigned long long *best, hipStream_t st) {
    argmax_degree_kernel<<<min(blocks_for(n, 256), 1024), 256, 0, st>>>(n, rp, best);
    return hipGetLastError();
}
hipError_t launch_sweep_update(int n, const int *dist, int *bound, int first, unsigned long long *far, hipStream_t st) {
    sweep_update_kernel<<<min(blocks_for(n, 256), 1024), 256, 0, st>>>(n, dist, bound, first, far);
    return hipGetLastError();
}
hipError_t launch_argmin_bound(int n, const int *bound, unsigned long long *best, hipStream_t st) {
    argmin_bound_kernel<<<min(blocks_for(n, 256), 1024), 256, 0, st>>>(n, bound, best);
    return hipGetLastError();
}
hipError_t launch_bfs_init(int n, int u, int *dist, int *parB, hipStream_t st) {
    bfs_init_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, u, dist, parB);
    return hipGetLastError();
}
static inline int row_grid(const RowMap &m, int G) {
    const long long tiles = ((long long)m.n + (256 / G) - 1) / (256 / G);
    return (int)std::min<long long>(std::max<long long>(tiles, 1), 4096);
}

hipError_t launch_bfs_level(const RowMap &m, int G, int d, int *dist, int *parB, int *found, const int *prev,
                            hipStream_t st) {
    const int grid = row_grid(m, G);
    USTD_DISPATCH_G(G, bfs_level_kernel<GG><<<grid, 256, 0, st>>>(m, d, dist, parB, found, prev));
    return hipGetLastError();
}
hipError_t launch_heavy_list(int n, const int *rp, int thresh, int *bcount, int *heavy, int *nheavy, hipStream_t st) {
    const int nb = blocks_for(n, 256);
    heavy_count_kernel<<<nb, 256, 0, st>>>(n, rp, thresh, bcount);
    heavy_scan_kernel<<<1, 256, 0, st>>>(nb, bcount, nheavy);
    heavy_write_kernel<<<nb, 256, 0, st>>>(n, rp, thresh, bcount, heavy);
    return hipGetLastError();
}
hipError_t launch_count_unreached(int n, const int *dist, int *err, hipStream_t st) {
    count_unreached_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, dist, err);
    return hipGetLastError();
}
template <bool LDS, typename CT, bool WT, bool BV = false>
int resident_of(size_t dyn, int *per_cu) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, wilson_kernel<LDS, CT, WT, false, BV>, 64, dyn) ==
           hipSuccess;
}
int wilson_resident_blocks(bool lds_bits, bool col16, bool weighted, int nwords, bool block_split) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const size_t dyn = lds_bits ? (size_t)nwords * 4 : 0;
    int ok;
    if (block_split) {
        if (lds_bits) ok = col16 ? resident_of<true, unsigned short, false, true>(dyn, &per_cu)
                                 : resident_of<true, int, false, true>(dyn, &per_cu);
        else ok = col16 ? resident_of<false, unsigned short, false, true>(0, &per_cu)
                        : resident_of<false, int, false, true>(0, &per_cu);
    } else if (lds_bits) {
        if (col16) ok = weighted ? resident_of<true, unsigned short, true>(dyn, &per_cu)
                                 : resident_of<true, unsigned short, false>(dyn, &per_cu);
        else ok = weighted ? resident_of<true, int, true>(dyn, &per_cu) : resident_of<true, int, false>(dyn, &per_cu);
    } else {
        if (col16) ok = weighted ? resident_of<false, unsigned short, true>(0, &per_cu)
                                 : resident_of<false, unsigned short, false>(0, &per_cu);
        else ok = weighted ? resident_of<false, int, true>(0, &per_cu) : resident_of<false, int, false>(0, &per_cu);
    }
    if (!ok) return 0;
    return std::max(1, per_cu) * std::max(1, cus);
}
long long wilson_graph_lds_bytes(int n, long long nnz, bool hops) {
    return ((long long)(n + 1) * 4 + (long long)n * 4 + (hops ? nnz * 4 : 0) + nnz * 2 + 3) / 4 * 4;
}
int wilson_resident_blocks_graph_lds(int nwords, long long graph_bytes) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    hipFuncAttributes fa{};
    if (hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(wilson_kernel<true, unsigned short, false, true>)) !=
        hipSuccess)
        return 0;
    const long long dyn = (long long)nwords * 4 + graph_bytes;
    const long long bytes = ((long long)fa.sharedSizeBytes + dyn + 255) / 256 * 256;
    if (bytes > 65536) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, wilson_kernel<true, unsigned short, false, true>, 64,
                                                     (size_t)dyn) != hipSuccess)
        return 0;
    const int by_lds = 2 * (int)(81920 / bytes);  // two 80 KB halves, whole blocks in each
    return std::max(0, std::min(per_cu, by_lds)) * std::max(1, cus);
}
template <bool LDS, typename CT>
void launch_wilson_t(const WilsonArgs &a, int blocks, bool weighted, bool bv, size_t dyn, hipStream_t st) {
    if (bv) wilson_kernel<LDS, CT, false, false, true><<<blocks, 64, dyn, st>>>(a);
    else if (weighted) wilson_kernel<LDS, CT, true><<<blocks, 64, dyn, st>>>(a);
    else wilson_kernel<LDS, CT, false><<<blocks, 64, dyn, st>>>(a);
}
hipError_t launch_wilson(const WilsonArgs &a, int blocks, bool lds_bits, bool col16, bool weighted, int nwords,
                         hipStream_t st, long long graph_lds_bytes, bool block_split) {
    if (block_split && (weighted || a.tiles || graph_lds_bytes > 0)) return hipErrorInvalidValue;
    if (graph_lds_bytes > 0) {
        if (!lds_bits || !col16 || weighted || a.tiles) return hipErrorInvalidValue;
        wilson_kernel<true, unsigned short, false, true>
            <<<blocks, 64, (size_t)nwords * 4 + (size_t)graph_lds_bytes, st>>>(a);
        return hipGetLastError();
    }
    if (lds_bits) {
        const size_t dyn = (size_t)nwords * 4;
        if (col16) launch_wilson_t<true, unsigned short>(a, blocks, weighted, block_split, dyn, st);
        else launch_wilson_t<true, int>(a, blocks, weighted, block_split, dyn, st);
    } else {
        if (col16) launch_wilson_t<false, unsigned short>(a, blocks, weighted, block_split, 0, st);
        else launch_wilson_t<false, int>(a, blocks, weighted, block_split, 0, st);
    }
    return hipGetLastError();
}
hipError_t launch_tree_records(const IntervalArgs &a, int ntrees, int *open, hipStream_t st) {
    int rounds = 1;  // 8^rounds >= n: then every path is covered (at most kTreeJumpRounds for n < 2^30)
    for (long long len = 8; len < a.n; len *= 8) ++rounds;
    if (a.n <= kTreeSmallMaxN) {
        tree_records_small_kernel<<<ntrees, 256, 0, st>>>(a, rounds);
        return hipGetLastError();
    }
    const dim3 grid(blocks_for(a.n, 256), ntrees);
    tree_jump_init_kernel<<<grid, 256, 0, st>>>(a, open);
    for (int r = 0; r < rounds; ++r) tree_jump_kernel<<<grid, 256, 0, st>>>(a, open + r);
    tree_records_kernel<<<grid, 256, 0, st>>>(a);
    return hipGetLastError();
}
hipError_t launch_extract_parents(int n, int ntrees, const int *rec, long long rec_stride, int *out, hipStream_t st) {
    // a dispatch counts its work-items in 32 bits: at most 2^31 (vertex, tree) items per launch
    const int chunk = (int)std::max(1ll, std::min<long long>(ntrees, (1ll << 31) / std::max(n, 1)));
    for (int t0 = 0; t0 < ntrees; t0 += chunk) {
        const int nt = std::min(chunk, ntrees - t0);
        extract_parents_kernel<<<blocks_for((long long)n * nt, 256), 256, 0, st>>>(
            n, nt, rec + (long long)t0 * 2 * rec_stride, rec_stride, out + (long long)t0 * n);
    }
    return hipGetLastError();
}
hipError_t launch_b_intervals(int n, int u, int ecc, const int *dist, const int *parB, int *scratch, int2 *bint,
                              int *bflag, hipStream_t st) {
    int *sz = scratch, *cur = scratch + n, *pre = scratch + 2 * n;
    const int nb = blocks_for(n, 256);
    bsub_init_kernel<<<nb, 256, 0, st>>>(n, u, sz, cur, pre);
    for (int d = ecc; d >= 1; --d) bsub_size_kernel<<<nb, 256, 0, st>>>(n, d, dist, parB, sz);
    for (int d = 1; d <= ecc; ++d) bsub_pre_kernel<<<nb, 256, 0, st>>>(n, d, dist, parB, sz, cur, pre);
    bsub_pack_kernel<<<nb, 256, 0, st>>>(n, parB, pre, sz, bint, bflag);
    return hipGetLastError();
}
hipError_t launch_sweep_small(const RowMap &m, int G, int sweeps, int *dist, int *bound, int *pivot, hipStream_t st) {
    USTD_DISPATCH_G(G, (sweep_small_kernel<GG><<<1, kSweepThreads, 0, st>>>(m, sweeps, dist, bound, pivot)));
    return hipGetLastError();
}
hipError_t launch_setup_small(const RowMap &m, int G, int u, int *dist, int *parB, int *scratch, int2 *bint,
                              int *bflag, int *out, hipStream_t st) {
    USTD_DISPATCH_G(G, (setup_small_kernel<GG><<<1, kSetupThreads, 0, st>>>(m, u, dist, parB, scratch, bint, bflag,
                                                                             out)));
    return hipGetLastError();
}
hipError_t launch_centralities(long long n, const double *diag, double *farness, double *closeness, double *nrwb,
                               double *scalars, hipStream_t st) {
    double *part = nullptr;  // an output that may hold the partial sums meanwhile
    if (n > kTraceOneMax) {
        const uintptr_t d0 = reinterpret_cast<uintptr_t>(diag), d1 = reinterpret_cast<uintptr_t>(diag + n);
        for (double *o : {farness, closeness, nrwb}) {
            const uintptr_t o0 = reinterpret_cast<uintptr_t>(o), o1 = reinterpret_cast<uintptr_t>(o + n);
            if (o && !part && (o1 <= d0 || d1 <= o0)) part = o;
        }
    }
    if (part) {
        const int nb = (int)((n + kTracePerBlock - 1) / kTracePerBlock);  // < n
        trace_partial_kernel<<<nb, 256, 0, st>>>(n, diag, part);
        trace_finish_kernel<<<1, kTraceThreads, 0, st>>>(n, nb, part, scalars);
    } else {
        trace_kernel<<<1, kTraceThreads, 0, st>>>(n, diag, scalars);
    }
    if (farness || closeness || nrwb)
        centrality_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, diag, scalars, farness, closeness, nrwb);
    return hipGetLastError();
}
hipError_t launch_edge_counts(const EdgeCountArgs &a, hipStream_t st) {
    dim3 grid(blocks_for(a.n, 256), (a.ntrees + a.trees_per_chunk - 1) / a.trees_per_chunk);
    edge_count_kernel<<<grid, 256, 0, st>>>(a);
    return hipGetLastError();
}
hipError_t launch_edge_fold(int n, long long nnz, const int *rp, const int *col, long long *counts, hipStream_t st) {
    edge_fold_kernel<<<blocks_for(nnz, 256), 256, 0, st>>>(n, nnz, rp, col, counts);
    return hipGetLastError();
}
template <int CH, int PL>
static void launch_aggregate_t(const AggregateArgs &a, hipStream_t st) {
    const dim3 grid(blocks_for(a.n, 256), (a.ntrees + CH - 1) / CH);
    if (a.F) aggregate_kernel<true, CH, PL><<<grid, 256, 0, st>>>(a);
    else aggregate_kernel<false, CH, PL><<<grid, 256, 0, st>>>(a);
}
template <int CH>
static void launch_aggregate_c(const AggregateArgs &a, hipStream_t st) {
    if (a.ecc >= 1 && a.ecc <= 5) launch_aggregate_t<CH, 4>(a, st);
    else if (a.ecc >= 1 && a.ecc <= 9) launch_aggregate_t<CH, 8>(a, st);
    else launch_aggregate_t<CH, 0>(a, st);
}
hipError_t launch_aggregate(const AggregateArgs &a, hipStream_t st) {
    if (a.chunk == kAggChunkLarge) launch_aggregate_c<kAggChunkLarge>(a, st);
    else launch_aggregate_c<kAggChunk>(a, st);
    return hipGetLastError();
}
__global__ void fill_i64_kernel(long long n, long long *__restrict__ a, long long v) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = v;
}
__global__ void add_i64_kernel(long long n, const long long *__restrict__ a, long long *__restrict__ b) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] += a[i];
}
hipError_t launch_fill_i64(long long n, long long *a, long long v, hipStream_t st) {
    if (n > 0) fill_i64_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, a, v);
    return hipGetLastError();
}
hipError_t launch_add_i64(long long n, const long long *a, long long *b, hipStream_t st) {
    if (n > 0) add_i64_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, a, b);
    return hipGetLastError();
}
hipError_t launch_edge_resistance(int n, long long nnz, const long long *rp, const int *col, const double *w,
                                  const long long *counts, double q, double theta, double *r, double *denom,
                                  hipStream_t st) {
    if (nnz > 0)
        edge_resistance_kernel<<<blocks_for(nnz, 256), 256, 0, st>>>(n, nnz, rp, col, w, counts, q, theta, r, denom);
    return hipGetLastError();
}
hipError_t launch_combine(int n, int u, double den, const long long *counts, const double *x, double *diag,
                          hipStream_t st) {
    combine_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, u, den, counts, x, diag);
    return hipGetLastError();
}
hipError_t launch_sum_walks(int cnt, const long long *steps, const long long *draws, unsigned long long *totals,
                            hipStream_t st) {
    sum_walks_kernel<<<1, 256, 0, st>>>(cnt, steps, draws, totals);
    return hipGetLastError();
}
hipError_t launch_tile_walks(int cnt, const WilsonTile *tiles, const long long *steps, const long long *draws,
                             unsigned long long *totals, hipStream_t st) {
    if (cnt > 0) tile_walks_kernel<<<blocks_for(cnt, 256), 256, 0, st>>>(cnt, tiles, steps, draws, totals);
    return hipGetLastError();
}
hipError_t launch_row_cumsum(int n, int nnz, const int *rp, const double *w, int heavy_thresh, const int *heavy,
                             const int *nheavy, double *cw, double *wdeg, int *guide, hipStream_t st) {
    row_cumsum_kernel<<<std::min(blocks_for(n, 256), 4096), 256, 0, st>>>(n, rp, w, heavy_thresh, cw, wdeg);
    row_cumsum_heavy_kernel<<<1024, kWave, 0, st>>>(rp, w, heavy, nheavy, cw, wdeg);
    step_guide_kernel<<<std::min(blocks_for(nnz, 256), 8192), 256, 0, st>>>(n, nnz, rp, cw, guide);
    return hipGetLastError();
}
__global__ void vertex_rows_kernel(int n, const int *__restrict__ rp, const int *__restrict__ bflag,
                                   int4 *__restrict__ vrow) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n) vrow[v] = make_int4(rp[v], rp[v + 1], bflag[v], 0);
}
hipError_t launch_vertex_rows(int n, const int *rp, const int *bflag, int4 *vrow, hipStream_t st) {
    vertex_rows_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, rp, bflag, vrow);
    return hipGetLastError();
}
__global__ void hops_kernel(long long nnz, const int *__restrict__ col, const int *__restrict__ rp,
                            unsigned long long *__restrict__ hops) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < nnz; i += (long long)gridDim.x * blockDim.x) {
        const int y = col[i];
        hops[i] = (uint32_t)rp[y] | ((unsigned long long)(uint32_t)(rp[y + 1] - rp[y]) << 32);
    }
}
hipError_t launch_hops(long long nnz, const int *col, const int *rp, unsigned long long *hops, hipStream_t st) {
    hops_kernel<<<(int)std::min<long long>(blocks_for(nnz, 256), 16384), 256, 0, st>>>(nnz, col, rp, hops);
    return hipGetLastError();
}
hipError_t launch_check_weights(int n, const int *rp, const int *col, const double *w, int *err, hipStream_t st) {
    check_weights_kernel<<<std::min(blocks_for(n, 256), 4096), 256, 0, st>>>(n, rp, col, w, err);
    return hipGetLastError();
}
hipError_t launch_bpath(int n, int u, const int *rp, const int *col, const double *w, const int *parB, double *wB,
                        unsigned long long *rmax_bits, hipStream_t st) {
    b_edge_weight_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, u, rp, col, w, parB, wB);
    bpath_resist_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, u, parB, wB, rmax_bits);
    return hipGetLastError();
}
hipError_t launch_fixed_weights(int n, int u, const double *wB, int shift, long long *F, hipStream_t st) {
    fixed_weights_kernel<<<blocks_for(n, 256), 256, 0, st>>>(n, u, wB, ldexp(1.0, shift), F);
    return hipGetLastError();
}
hipError_t launch_philox_words(uint32_t key0, uint32_t key1, long long t, int s, long long k0, long long count,
                               uint32_t *out, hipStream_t st) {
    philox_words_kernel<<<blocks_for(count, 256), 256, 0, st>>>(key0, key1, t, s, k0, count, out);
    return hipGetLastError();
}

}  // namespace ustd
