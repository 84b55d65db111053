// ustd_device.hpp -- device-side helpers for the gfx950 kernels (wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ustd {

constexpr int kWave = 64;

// Philox4x32-10 (Salmon et al., SC 2011): ten rounds of two 32x32->64 multiplies whose
// halves are mixed with the odd counter words and the key, the key advancing by the
// Weyl increments between rounds.
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // full 32x32 -> 64-bit products: one v_mad_u64_u32 each instead of a low and a high multiply
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c.z;
        c = make_uint4((uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1, (uint32_t)p0);
    }
    return c;
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int l = lane_id();
    return l ? (~0ull >> (64 - l)) : 0ull;
}

// inclusive prefix sum across the 64 lanes of a wave
template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
    const int l = lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        T o = __shfl_up(v, d, kWave);
        if (l >= d) v += o;
    }
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

// Block-wide inclusive scan of one int per thread; *total receives the block sum.
// `sh` must hold at least blockDim.x / 64 + 1 ints.  Contains two barriers.
__device__ __forceinline__ int block_incl_scan(int v, int *total, int *sh) {
    const int l = lane_id(), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    int incl = wave_incl_scan(v);
    if (l == kWave - 1) sh[w] = incl;
    __syncthreads();
    int off = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        const int s = sh[i];
        off += (i < w) ? s : 0;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return incl + off;
}

// Block-wide sum of doubles in a fixed order (deterministic for a fixed blockDim).
__device__ __forceinline__ double block_sum(double v, double *sh) {
    const int l = lane_id(), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    v = wave_sum(v);
    if (l == 0) sh[w] = v;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < nw; ++i) s += sh[i];
    __syncthreads();
    return s;
}

// Block-wide sum of one value per thread in a fixed order (deterministic for a fixed number of
// threads nt: the block, or its first nt threads when the others have left the kernel);
// `sh` holds at least nt / 64 values.  Contains two barriers.
template <typename T>
__device__ __forceinline__ T block_sum_t(T v, T *sh, int nt) {
    const int l = lane_id(), w = threadIdx.x / kWave, nw = nt / kWave;
    v = wave_sum(v);
    if (l == 0) sh[w] = v;
    __syncthreads();
    T s = (T)0;
    for (int i = 0; i < nw; ++i) s += sh[i];
    __syncthreads();
    return s;
}
template <typename T>
__device__ __forceinline__ T block_sum_t(T v, T *sh) {
    return block_sum_t<T>(v, sh, (int)blockDim.x);
}

// A record's word holds a vertex in 30 bits, whose largest value marks a free vertex: the vertices of a
// graph (the slots of a block-split graph) that the sampler takes.
constexpr int kFree = 0x3FFFFFFF;
__host__ __device__ __forceinline__ bool ids_fit(long long count) { return count < kFree; }

// Walk steps and draws of a tree: a lane of its wave counts in 32 bits, the wave (uniform) in 64.
//   steps: the walks that a lane commits in batches, at most kBatchSteps a start, are the lane's, and a
//   tree has fewer than 2^30 starts; what the wave commits together is the wave's, but for a tree
//   within the LDS bitmap, where 2^17 starts of kWalkDraws steps fit lane 0's counter (the wave's costs
//   the graph-in-LDS sampler 4% on long lone walks: six more scalar registers spilled);
//   draws: at most kWalkDraws a start that the lane walks, moved to the wave's counter once every
//   kDrawWindow starts of the tree (another kDrawWindow bounds the starts then in flight).
constexpr unsigned kBatchSteps = 4, kWalkDraws = 250, kDrawWindow = 1u << 22;
static_assert((1ull << 30) * kBatchSteps <= 1ull << 32, "a lane's batch commits fit");
static_assert((1ull << 17) * (kWalkDraws + kBatchSteps) < 1ull << 32, "all commits within the bitmap fit a lane");
static_assert(2ull * kDrawWindow * kWalkDraws < 1ull << 32, "a lane's draws between two moves fit");

// of a walk of k steps that the wave committed: the lane's part, the wave's part
template <bool LDS>
__host__ __device__ __forceinline__ uint32_t long_walk_lane(int k, int lane) { return LDS && lane == 0 ? (uint32_t)k : 0u; }
template <bool LDS>
__host__ __device__ __forceinline__ long long long_walk_wave(int k) { return LDS ? 0 : k; }
// whether the lanes' draws move before the window of starts at `start`
__host__ __device__ __forceinline__ bool draws_move(int start) {
    return start != 0 && (start & (int)(kDrawWindow - 1)) == 0;
}

// Threads at work in the one-workgroup solve.  Where the rows' lane groups fill less than the
// workgroup, four waves do the work and the others leave at once (a barrier counts the waves that
// are left): an iteration is a chain of a dozen barriers, which cost less among four (column of a
// 13 x 11 grid 306 us against 333, 8 x 8 grid 267 against 279).  Beyond that the product grows by more than the barriers save: 20 x 30 grid 1643 us
// against 1109, R-MAT scale 10 1709 against 764.  The choice depends on the graph alone, so a batch
// member's solve is that of a single call.
constexpr int kSmallThreads = 1024, kFewThreads = 256;
__host__ __device__ __forceinline__ int small_solve_threads(int n, int G) {
    return (long long)n * G < kSmallThreads ? kFewThreads : kSmallThreads;
}

// ---- CSR rows.  Slots are below 2^31 (nnz < 2^31), and a loop over a row in strides looks past the
// row's end by up to a stride, so it counts in unsigned slots: a row that ends just below 2^31 does
// not wrap.  (Host code too: the tests walk such rows on the CPU.)

// The sum of two slots takes 32 bits unsigned (rows behind slot 2^30).
__host__ __device__ __forceinline__ int mid_slot(int lo, int hi) { return (int)(((uint32_t)lo + (uint32_t)hi) >> 1); }

// first slot of the ascending row [lo, hi) whose column is x or above (hi: none)
__host__ __device__ __forceinline__ int row_lower_bound(const int *__restrict__ col, int lo, int hi, int x) {
    while (lo < hi) {
        const int mid = mid_slot(lo, hi);
        if (col[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// slot of x in the ascending row [lo, hi), or -1
__host__ __device__ __forceinline__ int find_in_row(const int *__restrict__ col, int lo, int hi, int x) {
    while (lo < hi) {
        const int mid = mid_slot(lo, hi);
        const int c = col[mid];
        if (c == x) return mid;
        if (c < x) lo = mid + 1;
        else hi = mid;
    }
    return -1;
}

// f(slot) for the slots lo + first, lo + first + step, ... below hi
template <typename F>
__host__ __device__ __forceinline__ void row_each(int lo, int hi, uint32_t first, uint32_t step, F f) {
    const uint32_t end = (uint32_t)hi;
    for (uint32_t e = (uint32_t)lo + first; e < end; e += step) f(e);
}

// run = the sum of w[lo .. hi) from left to right, cw[e] the sums up to each entry
__host__ __device__ __forceinline__ double row_running_sums(const double *__restrict__ w, double *__restrict__ cw,
                                                            int lo, int hi) {
    double run = 0.0;
    int e = lo;
    for (; hi - e >= 8; e += 8) {  // eight loads in flight, the additions still in order
        double wv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) wv[k] = w[e + k];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            run += wv[k];
            cw[e + k] = run;
        }
    }
    for (; e < hi; ++e) {
        run += w[e];
        cw[e] = run;
    }
    return run;
}

// acc + sum of the entries lo + first, lo + first + step, ... below hi, in that order, U loads at a
// time; weighted entries with w
template <typename T, int U>
__host__ __device__ __forceinline__ T row_sum(T acc, const int *__restrict__ col, const double *__restrict__ w,
                                              const T *__restrict__ p, int lo, int hi, uint32_t first, uint32_t step) {
    const uint32_t end = (uint32_t)hi;
    for (uint32_t e = (uint32_t)lo + first; e < end; e += U * step) {
        int c[U];
        T q[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            c[k] = -1;
            if (e + k * step < end) c[k] = col[e + k * step];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            q[k] = (T)0;
            if (c[k] >= 0) q[k] = w ? (T)w[e + k * step] * p[c[k]] : p[c[k]];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) acc += q[k];
    }
    return acc;
}

}  // namespace ustd
