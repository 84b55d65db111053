// ustd_solve.hip -- the pivot-column solve of the UST estimator of diag(L^+) on gfx950:
// L x = e_u - (1/n) 1 with x orthogonal to 1, which is column u of L^+ (Section "Overview",
// step 1; Algorithm 1, solver accuracy eta).  The paper solves it with conjugate gradients
// and the diagonal (Jacobi) preconditioner (Appendix "UST Generation, Pivot Selection, and
// the Linear System").
//
// Here CG runs with reliable updates: the solution x is accumulated in FP64, while the
// iteration itself runs on vectors of type T, FP64 or (mixed mode) FP32: the correction xs
// since the last update, the iterated residual rs, z = rs / diag, the direction p and q = L p.
// A reliable update folds xs into x and replaces rs by the true residual b - L x computed in
// FP64, keeping the direction p, so the Krylov space is not thrown away.  It is taken when
// |rs| has dropped by a factor delta since the largest residual after the previous update,
// when |rs| reaches the target, or at the iteration cap; the solve ends at an update whose
// true residual meets the target.  Dot products are accumulated in FP64 in a fixed order.
//
// Two engines: the whole solve in one workgroup (small graphs; many graphs of a batch side by
// side, one workgroup each), with no host round trip; or three kernels per slot whose scalars
// stay on the device, enqueued by the host in growing chunks ahead of a `done` flag that turns
// later launches into no-ops.  A slot is one CG iteration or the second half of a reliable update.
#include "ustd_kernels.hpp"

#include <algorithm>

namespace ustd {

// blocks of the multi-kernel engine: at most one resident set (8 per compute unit), since every
// block adds a ticket and a partial result to its kernel's tail
constexpr int kSolveGrid = 2048;
static_assert(kSolveGrid <= kMaxSolveGrid, "partial results fit the workspace");

// y = L p over all rows, degree-balanced: rows of degree <= heavy_thresh by groups of G lanes,
// heavier rows (listed in ascending order) by the whole block.  emit(v, (L p)_v) is called once
// per row from one thread.  Fixed grid and fixed per-row reduction trees: deterministic.
// Block blk of nblk takes every nblk-th heavy row and row tile (a whole grid: blockIdx.x of
// gridDim.x; a workgroup that solves a graph alone: 0 of 1).  BS = block size.
// A row is a chain of three loads (row bounds, columns, the gathered entries), so what bounds the
// product is how many chains are in flight: a group takes the first two entries a lane of
// kRowsInFlight rows at once, then what is left of the longer rows four entries a lane at a time,
// and a heavy row goes eight entries a thread at a time.  (One entry at a time, a light row of
// degree 512 is 32 loads in a row, longer than the rest of the product at n = 200k, and the hub of
// R-MAT scale 22 kept one workgroup busy for 1.0 ms of a 1.2 ms product.)
constexpr int kRowsInFlight = 4;

// the light rows; R rows of a group in flight
template <typename T, int G, int R, typename Emit>
__device__ __forceinline__ void lap_light_rows(const RowMap &m, const T *__restrict__ p, Emit emit, int blk, int nblk,
                                               int bs) {
    const double *__restrict__ w = m.w;
    const int rows_per_tile = bs / G;
    const int g = threadIdx.x / G, l = threadIdx.x % G;
    for (int tile = blk; tile * rows_per_tile < m.n; tile += R * nblk) {
        int lo[R], deg[R], len[R];
        int c[R][2];
        T q[R][2];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int v = (tile + i * nblk) * rows_per_tile + g;
            lo[i] = v < m.n ? m.rp[v] : 0;
            deg[i] = v < m.n ? m.rp[v + 1] : -1;
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            deg[i] = deg[i] < 0 ? -1 : deg[i] - lo[i];
            len[i] = deg[i] <= m.heavy_thresh ? deg[i] : 0;  // heavy rows are done above
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                c[i][s] = -1;
                if (l + s * G < len[i]) c[i][s] = m.col[lo[i] + l + s * G];
            }
        }
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                q[i][s] = (T)0;
                if (c[i][s] >= 0) q[i][s] = w ? (T)w[lo[i] + l + s * G] * p[c[i][s]] : p[c[i][s]];
            }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if ((tile + i * nblk) * rows_per_tile >= m.n) break;  // no row left for any group
            T acc = q[i][0] + q[i][1];
            if (len[i] > 2 * G) acc = row_sum<T, 4>(acc, m.col, w, p, lo[i], lo[i] + len[i], l + 2 * G, G);
#pragma unroll
            for (int dd = G / 2; dd > 0; dd >>= 1) acc += __shfl_xor(acc, dd, G);
            if (deg[i] >= 0 && deg[i] <= m.heavy_thresh && l == 0) {
                const int v = (tile + i * nblk) * rows_per_tile + g;
                emit(v, (w ? (T)m.wdeg[v] : (T)deg[i]) * p[v] - acc);
            }
        }
    }
}

template <typename T, int G, int BS = 256, typename Emit>
__device__ __forceinline__ void lap_apply_rows(const RowMap &m, const T *__restrict__ p, Emit emit, int blk,
                                               int nblk, int bs = BS) {
    __shared__ T shr[BS / kWave];
    const int nh = *m.nheavy;
    const double *__restrict__ w = m.w;  // uniform: weighted Laplacian when set
    for (int h = blk; h < nh; h += nblk) {
        const int v = m.heavy[h];
        const int lo = m.rp[v], hi = m.rp[v + 1];
        T acc = row_sum<T, 8>((T)0, m.col, w, p, lo, hi, threadIdx.x, bs);
        acc = block_sum_t<T>(acc, shr, bs);
        if (threadIdx.x == 0) emit(v, (w ? (T)m.wdeg[v] : (T)(hi - lo)) * p[v] - acc);
    }
    if (m.n <= bs / G) lap_light_rows<T, G, 1>(m, p, emit, blk, nblk, bs);  // one row a group at most: four in flight cost 4% there (16 x 16 grid)
    else lap_light_rows<T, G, kRowsInFlight>(m, p, emit, blk, nblk, bs);
}

// Jacobi diagonal: the degree, or the conductance sum of a weighted Laplacian's row
template <typename T>
__device__ __forceinline__ T jacobi_diag(const SolveArgs<T> &a, int v) {
    return a.wdeg ? (T)a.wdeg[v] : (T)(a.rp[v + 1] - a.rp[v]);
}

// right-hand side e_u - 1/n
__device__ __forceinline__ double rhs_of(int v, int u, double inv_n) { return (v == u ? 1.0 : 0.0) - inv_n; }

// Sum of per-block partials part[i * stride], i < nparts, in index order by one block.
__device__ __forceinline__ double sum_partials(const double *__restrict__ part, int nparts, int stride, double *sh) {
    double v = 0.0;
    for (int i = threadIdx.x; i < nparts; i += blockDim.x) v += part[(long long)i * stride];
    return block_sum(v, sh);
}

// partial regions: p.q | (z.r, r.r) of the update | (z.r, |b - L x|^2) of a reliable update
__device__ __forceinline__ double *part_pq(double *part) { return part; }
__device__ __forceinline__ double *part_upd(double *part) { return part + kMaxSolveGrid; }
__device__ __forceinline__ double *part_rel(double *part) { return part + 3 * kMaxSolveGrid; }

// The last block of a grid to finish sums the blocks' partial results, so a reduction needs no
// kernel of its own.  The blocks run on several XCDs whose L2s are not coherent within a kernel:
// partial results are stored past the L2 (agent scope), the store is complete before the block
// takes its ticket, and the last block reads them past the L2.  Tickets on one address cost 14 ns
// each (2048 blocks: 28 us), so block b takes one of group b mod kTicketGroups (its own cache
// line), and the last of a group one of the root.  Thread 0 stores and takes tickets; every
// thread learns the answer.  The counters are left at zero.
constexpr int kTicketGroups = 32, kTicketStride = 32;  // counters a 128-byte line apart
static_assert(2 * kSolveGrid + (kTicketGroups + 1) * kTicketStride / 2 <= 2 * kMaxSolveGrid, "counters fit beside the partials");
__device__ __forceinline__ unsigned *part_tickets(double *part) {  // behind the partials of the update
    return reinterpret_cast<unsigned *>(part_upd(part) + 2 * kSolveGrid);
}
__device__ __forceinline__ void put_partial(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool take_ticket(unsigned *t, unsigned of) {
    const bool last = __hip_atomic_fetch_add(t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == of - 1;
    if (last) __hip_atomic_store(t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last;
}
__device__ __forceinline__ bool last_block(double *part) {
    __shared__ int last;
    if (threadIdx.x == 0) {
        unsigned *t = part_tickets(part);
        const unsigned groups = min(gridDim.x, (unsigned)kTicketGroups), g = blockIdx.x % groups;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the partial results have been stored
        last = 0;
        if (take_ticket(t + g * kTicketStride, (gridDim.x - g + groups - 1) / groups))
            last = take_ticket(t + kTicketGroups * kTicketStride, groups);
    }
    __syncthreads();
    return last;
}
// sums of part[N i + j], i < nparts (at most kSolveGrid), j < N, into out[j], in the order of
// sum_partials; every load is issued before the first is waited for
template <int N>
__device__ __forceinline__ void sum_fresh(double *part, int nparts, double *out, double *sh) {
    constexpr int kEach = kSolveGrid / 256;
    double v[kEach][N];
#pragma unroll
    for (int k = 0; k < kEach; ++k)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int i = threadIdx.x + k * 256;
            v[k][j] = 0.0;
            if (i < nparts)
                v[k][j] = __hip_atomic_load(&part[(long long)N * i + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < kEach; ++k) s += v[k][j];
        out[j] = block_sum(s, sh);
    }
}

// ---------------------------------------------------------------------------------------
// multi-kernel solve (large graphs): three kernels per slot, whose scalars stay on the device; once
// `done` is set every later launch of the solve returns at once.  With a kernel per reduction and
// per half of an update (eight an iteration, five of them a few microseconds of launch for next
// to no work) the pivot column of a hyperbolic graph with n = 200k (about 700 iterations) took 50.9 ms;
// now 34.6.  Medians there: the product 34 us (4 million gathers, each a line through the L2), the
// update 9, the direction 5.
// ---------------------------------------------------------------------------------------
// x = 0, xs = 0, rs = b, z = p = rs / diag; partials of z.r, r.r and b.b (3 per block)
template <typename T>
__global__ __launch_bounds__(256) void solve_start_kernel(SolveArgs<T> a) {
    __shared__ double sh[4];
    const double inv_n = 1.0 / (double)a.n;
    double rz = 0.0, rr = 0.0, bb = 0.0;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n; v += gridDim.x * blockDim.x) {
        const double b = rhs_of(v, a.u, inv_n);
        const T rv = (T)b;
        const T zv = rv / jacobi_diag(a, v);
        a.x[v] = 0.0;
        a.xs[v] = (T)0;
        a.rs[v] = rv;
        a.z[v] = zv;
        a.p[v] = zv;
        rz += (double)rv * (double)zv;
        rr += (double)rv * (double)rv;
        bb += b * b;
    }
    rz = block_sum(rz, sh);
    rr = block_sum(rr, sh);
    bb = block_sum(bb, sh);
    if (threadIdx.x == 0) {
        double *pr = part_rel(a.part) + 3 * blockIdx.x;
        pr[0] = rz;
        pr[1] = rr;
        pr[2] = bb;
    }
}

template <typename T>
__global__ __launch_bounds__(256) void solve_start_finish_kernel(SolveArgs<T> a, double tol2, double delta2,
                                                                 int maxit) {
    __shared__ double sh[4];
    const double *pr = part_rel(a.part);
    for (int i = threadIdx.x; i < (kTicketGroups + 1) * kTicketStride; i += blockDim.x) part_tickets(a.part)[i] = 0u;
    const double rz = sum_partials(pr, a.grid_vec, 3, sh);
    const double rr = sum_partials(pr + 1, a.grid_vec, 3, sh);
    const double bb = sum_partials(pr + 2, a.grid_vec, 3, sh);
    if (threadIdx.x == 0) {
        SolveScalars *S = a.sc;
        S->rz = rz;
        S->alpha = S->beta = 0.0;
        S->rr = rr;
        S->rr_max = rr;
        S->rr_true = bb;
        S->bb = bb;
        S->tol2 = tol2;
        S->delta2 = delta2;
        S->iter = 0;
        S->maxit = maxit;
        S->upd = 0;
        S->skip = 0;
        S->updates = 0;
        S->stalls = 0;
        S->broke = 0;
        S->done = (bb > 0.0 && rz > 0.0 && maxit > 0) ? 0 : 1;
    }
}

// First kernel of a slot.  An iteration: q = L p, and the last block alpha = z.r / p.q (a
// breakdown, p.q not positive, ends the solve at the next update).  After a fold: the second half
// of a reliable update, r = b - L x in FP64, rs = r, z = rs / diag, and the last block decides on
// the true residual whether the solve ends, else beta from the replaced residual.  Three updates in
// a row whose true residual fell by less than 2x (the rounding floor) also end the solve.
template <typename T, int G>
__global__ __launch_bounds__(256) void solve_apply_kernel(SolveArgs<T> a, RowMap m) {
    __shared__ double sh[4];
    SolveScalars *S = a.sc;
    if (S->done) return;  // uniform: written by an earlier kernel
    if (!S->upd) {
        double acc = 0.0;
        T *__restrict__ q = a.q;
        const T *__restrict__ p = a.p;
        lap_apply_rows<T, G>(
            m, p,
            [&](int v, T qv) {
                q[v] = qv;
                acc += (double)p[v] * (double)qv;
            },
            blockIdx.x, gridDim.x);
        acc = block_sum(acc, sh);
        if (threadIdx.x == 0) put_partial(part_pq(a.part) + blockIdx.x, acc);
        if (!last_block(a.part)) return;
        double pq;
        sum_fresh<1>(part_pq(a.part), gridDim.x, &pq, sh);
        if (threadIdx.x == 0) {
            S->skip = 0;
            if (pq > 0.0 && pq == pq) {
                S->alpha = S->rz / pq;
            } else {
                S->alpha = 0.0;
                S->broke = 1;
            }
        }
        return;
    }
    const double inv_n = 1.0 / (double)a.n;
    double rz = 0.0, rt = 0.0;
    lap_apply_rows<double, G>(
        m, a.x,
        [&](int v, double lx) {
            const double rv = rhs_of(v, a.u, inv_n) - lx;
            const T rs = (T)rv;
            const T zv = rs / jacobi_diag(a, v);
            a.rs[v] = rs;
            a.z[v] = zv;
            rz += (double)rs * (double)zv;
            rt += rv * rv;
        },
        blockIdx.x, gridDim.x);
    rz = block_sum(rz, sh);
    rt = block_sum(rt, sh);
    double *pr = part_rel(a.part);
    if (threadIdx.x == 0) {
        put_partial(pr + 2 * blockIdx.x, rz);
        put_partial(pr + 2 * blockIdx.x + 1, rt);
    }
    if (!last_block(a.part)) return;
    double tot[2];
    sum_fresh<2>(pr, gridDim.x, tot, sh);
    const double rzn = tot[0];
    rt = tot[1];
    if (threadIdx.x == 0) {
        S->updates += 1;
        S->stalls = rt > 0.25 * S->rr_true ? S->stalls + 1 : 0;
        S->rr_true = rt;
        S->rr_max = rt;
        S->rr = rt;
        S->upd = 0;
        S->skip = 1;
        if (!(rt > S->tol2 * S->bb) || S->iter >= S->maxit || S->broke || S->stalls >= 3) {
            S->done = 1;
        } else {
            S->beta = S->rz != 0.0 ? rzn / S->rz : 0.0;
            S->rz = rzn;
        }
    }
}

// Second kernel of a slot, iterations only: xs += alpha p; rs -= alpha q; z = rs / diag; the last
// block counts the iteration and tests for a reliable update, else beta
template <typename T>
__global__ __launch_bounds__(256) void solve_update_kernel(SolveArgs<T> a) {
    __shared__ double sh[4];
    SolveScalars *S = a.sc;
    if (S->done || S->skip) return;
    const T al = (T)S->alpha;
    double rz = 0.0, rr = 0.0;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n; v += gridDim.x * blockDim.x) {
        a.xs[v] += al * a.p[v];
        const T rv = a.rs[v] - al * a.q[v];
        a.rs[v] = rv;
        const T zv = rv / jacobi_diag(a, v);
        a.z[v] = zv;
        rz += (double)rv * (double)zv;
        rr += (double)rv * (double)rv;
    }
    rz = block_sum(rz, sh);
    rr = block_sum(rr, sh);
    double *pu = part_upd(a.part);
    if (threadIdx.x == 0) {
        put_partial(pu + 2 * blockIdx.x, rz);
        put_partial(pu + 2 * blockIdx.x + 1, rr);
    }
    if (!last_block(a.part)) return;
    double tot[2];
    sum_fresh<2>(pu, gridDim.x, tot, sh);
    const double rzn = tot[0];
    rr = tot[1];
    if (threadIdx.x == 0) {
        S->iter += 1;
        S->rr = rr;
        const bool upd = S->broke || S->iter >= S->maxit || !(rr > S->tol2 * S->bb) || rr < S->delta2 * S->rr_max;
        if (rr > S->rr_max) S->rr_max = rr;
        S->upd = upd ? 1 : 0;
        if (!upd) {
            S->beta = S->rz != 0.0 ? rzn / S->rz : 0.0;
            S->rz = rzn;
        }
    }
}

// Third kernel of a slot: p = z + beta p, or the first half of a reliable update, x += xs, xs = 0
template <typename T>
__global__ __launch_bounds__(256) void solve_direction_kernel(SolveArgs<T> a) {
    if (a.sc->done) return;
    if (a.sc->upd) {
        for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n; v += gridDim.x * blockDim.x) {
            a.x[v] += (double)a.xs[v];
            a.xs[v] = (T)0;
        }
        return;
    }
    const T be = (T)a.sc->beta;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < a.n; v += gridDim.x * blockDim.x)
        a.p[v] = a.z[v] + be * a.p[v];
}

// ---------------------------------------------------------------------------------------
// the whole solve in one workgroup (small graphs, batch members): the same start, iteration,
// reliable updates and end rule, with no kernel boundary or host poll between iterations.
// Ends with the scalars the multi-kernel path leaves.
// ---------------------------------------------------------------------------------------
template <typename T, int G>
__device__ void solve_small_body(const SolveArgs<T> &a, const RowMap &m, double tol2, double delta2, int maxit,
                                 double *sh) {
    const int n = a.n, tid = threadIdx.x, u = a.u;
    const int nt = small_solve_threads(n, G);
    if (tid >= nt) return;
    const double inv_n = 1.0 / (double)n;
    double rz = 0.0, rr = 0.0, bb = 0.0;
    for (int v = tid; v < n; v += nt) {
        const double b = rhs_of(v, u, inv_n);
        const T rv = (T)b;
        const T zv = rv / jacobi_diag(a, v);
        a.x[v] = 0.0;
        a.xs[v] = (T)0;
        a.rs[v] = rv;
        a.z[v] = zv;
        a.p[v] = zv;
        rz += (double)rv * (double)zv;
        rr += (double)rv * (double)rv;
        bb += b * b;
    }
    rz = block_sum_t<double>(rz, sh, nt);  // the barriers also publish p before the first product
    rr = block_sum_t<double>(rr, sh, nt);
    bb = block_sum_t<double>(bb, sh, nt);
    double rr_max = rr, rr_true = bb;
    int it = 0, updates = 0, stalls = 0;
    bool done = !(bb > 0.0 && rz > 0.0 && maxit > 0);
    while (!done) {
        double pq = 0.0;
        lap_apply_rows<T, G, kSmallThreads>(
            m, a.p,
            [&](int v, T qv) {
                a.q[v] = qv;
                pq += (double)a.p[v] * (double)qv;
            },
            0, 1, nt);
        pq = block_sum_t<double>(pq, sh, nt);
        const bool broke = !(pq > 0.0 && pq == pq);
        const T al = broke ? (T)0 : (T)(rz / pq);
        double rzn = 0.0, rrn = 0.0;
        for (int v = tid; v < n; v += nt) {
            a.xs[v] += al * a.p[v];
            const T rv = a.rs[v] - al * a.q[v];
            a.rs[v] = rv;
            const T zv = rv / jacobi_diag(a, v);
            a.z[v] = zv;
            rzn += (double)rv * (double)zv;
            rrn += (double)rv * (double)rv;
        }
        rzn = block_sum_t<double>(rzn, sh, nt);
        rrn = block_sum_t<double>(rrn, sh, nt);
        ++it;
        const bool upd = broke || it >= maxit || !(rrn > tol2 * bb) || rrn < delta2 * rr_max;
        if (rrn > rr_max) rr_max = rrn;
        double beta;
        if (upd) {
            for (int v = tid; v < n; v += nt) {
                a.x[v] += (double)a.xs[v];
                a.xs[v] = (T)0;
            }
            __syncthreads();  // x complete before the product gathers it
            double rz2 = 0.0, rt = 0.0;
            lap_apply_rows<double, G, kSmallThreads>(
                m, a.x,
                [&](int v, double lx) {
                    const double rv = rhs_of(v, u, inv_n) - lx;
                    const T rs = (T)rv;
                    const T zv = rs / jacobi_diag(a, v);
                    a.rs[v] = rs;
                    a.z[v] = zv;
                    rz2 += (double)rs * (double)zv;
                    rt += rv * rv;
                },
                0, 1, nt);
            rz2 = block_sum_t<double>(rz2, sh, nt);
            rt = block_sum_t<double>(rt, sh, nt);
            ++updates;
            stalls = rt > 0.25 * rr_true ? stalls + 1 : 0;
            rr_true = rt;
            rr_max = rt;
            if (!(rt > tol2 * bb) || it >= maxit || broke || stalls >= 3) break;
            beta = rz != 0.0 ? rz2 / rz : 0.0;
            rz = rz2;
        } else {
            beta = rz != 0.0 ? rzn / rz : 0.0;
            rz = rzn;
        }
        const T be = (T)beta;
        for (int v = tid; v < n; v += nt) a.p[v] = a.z[v] + be * a.p[v];
        __syncthreads();  // p complete before the next product gathers it
    }
    if (tid == 0) {
        SolveScalars *S = a.sc;
        S->rz = rz;
        S->rr = rr_true;
        S->rr_max = rr_max;
        S->rr_true = rr_true;
        S->bb = bb;
        S->tol2 = tol2;
        S->delta2 = delta2;
        S->iter = it;
        S->maxit = maxit;
        S->upd = 0;
        S->updates = updates;
        S->stalls = stalls;
        S->done = 1;
    }
}

template <typename T, int G>
__global__ __launch_bounds__(kSmallThreads) void solve_small_kernel(SolveArgs<T> a, RowMap m, double tol2,
                                                                    double delta2, int maxit) {
    __shared__ double sh[kSmallThreads / kWave];
    solve_small_body<T, G>(a, m, tol2, delta2, maxit, sh);
}

// independent solves side by side: workgroup i runs job i (one graph's pivot column)
template <typename T, int G>
__global__ __launch_bounds__(kSmallThreads) void solve_small_batch_kernel(const SolveJob<T> *__restrict__ jobs) {
    __shared__ double sh[kSmallThreads / kWave];
    const SolveJob<T> &j = jobs[blockIdx.x];
    solve_small_body<T, G>(j.a, j.m, j.tol2, j.delta2, j.maxit, sh);
}

// ---------------------------------------------------------------------------------------
// final residual and projection
// ---------------------------------------------------------------------------------------
// res = b - L x (nullable), per-block partials of [sum res, |res|^2, sum x]; reduce3_kernel
// sums them into out[0..3)
template <int G>
__global__ __launch_bounds__(256) void residual64_kernel(RowMap m, int u, const double *__restrict__ x,
                                                         double *__restrict__ res, double *__restrict__ part) {
    __shared__ double sh[4];
    const double inv_n = 1.0 / (double)m.n;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    lap_apply_rows<double, G>(
        m, x,
        [&](int v, double lx) {
            const double rv = rhs_of(v, u, inv_n) - lx;
            if (res) res[v] = rv;
            s0 += rv;
            s1 += rv * rv;
            s2 += x[v];
        },
        blockIdx.x, gridDim.x);
    s0 = block_sum(s0, sh);
    s1 = block_sum(s1, sh);
    s2 = block_sum(s2, sh);
    if (threadIdx.x == 0) {
        part[blockIdx.x * 3] = s0;
        part[blockIdx.x * 3 + 1] = s1;
        part[blockIdx.x * 3 + 2] = s2;
    }
}

__global__ __launch_bounds__(256) void reduce3_kernel(const double *__restrict__ part, int nparts,
                                                      double *__restrict__ out) {
    __shared__ double sh[4];
    const double a0 = sum_partials(part, nparts, 3, sh);
    const double a1 = sum_partials(part + 1, nparts, 3, sh);
    const double a2 = sum_partials(part + 2, nparts, 3, sh);
    if (threadIdx.x == 0) {
        out[0] = a0;
        out[1] = a1;
        out[2] = a2;
    }
}

// x -= mean_src[0] / n (mean-zero projection)
__global__ __launch_bounds__(256) void project_kernel(int n, double *__restrict__ x,
                                                     const double *__restrict__ mean_src) {
    const double mean = mean_src[0] / (double)n;
    for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) x[v] -= mean;
}

// ---------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------
int solve_grid(const RowMap &m, int G) {
    const long long tiles = ((long long)m.n + (256 / G) - 1) / (256 / G);
    const long long blocks = (tiles + kRowsInFlight - 1) / kRowsInFlight;
    return (int)std::min<long long>(std::max<long long>(blocks, 1), kSolveGrid);
}
int vec_grid(int n) { return std::max(1, std::min((n + 255) / 256, kSolveGrid)); }

template <typename T>
hipError_t launch_solve_start(const SolveArgs<T> &a, double tol2, double delta2, int maxit, hipStream_t st) {
    solve_start_kernel<T><<<a.grid_vec, 256, 0, st>>>(a);
    solve_start_finish_kernel<T><<<1, 256, 0, st>>>(a, tol2, delta2, maxit);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_solve_slot(const SolveArgs<T> &a, const RowMap &m, int G, hipStream_t st) {
    USTD_DISPATCH_G(G, (solve_apply_kernel<T, GG><<<a.grid_spmv, 256, 0, st>>>(a, m)));
    solve_update_kernel<T><<<a.grid_vec, 256, 0, st>>>(a);
    solve_direction_kernel<T><<<a.grid_vec, 256, 0, st>>>(a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_solve_small(const SolveArgs<T> &a, const RowMap &m, int G, double tol2, double delta2, int maxit,
                              hipStream_t st) {
    USTD_DISPATCH_G(G, (solve_small_kernel<T, GG><<<1, kSmallThreads, 0, st>>>(a, m, tol2, delta2, maxit)));
    return hipGetLastError();
}

template <typename T>
hipError_t launch_solve_small_batch(const SolveJob<T> *jobs, int count, int G, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    USTD_DISPATCH_G(G, (solve_small_batch_kernel<T, GG><<<count, kSmallThreads, 0, st>>>(jobs)));
    return hipGetLastError();
}

#define USTD_SOLVE_INSTANTIATE(T)                                                                              \
    template hipError_t launch_solve_start<T>(const SolveArgs<T> &, double, double, int, hipStream_t);         \
    template hipError_t launch_solve_slot<T>(const SolveArgs<T> &, const RowMap &, int, hipStream_t);          \
    template hipError_t launch_solve_small<T>(const SolveArgs<T> &, const RowMap &, int, double, double, int,  \
                                              hipStream_t);                                                    \
    template hipError_t launch_solve_small_batch<T>(const SolveJob<T> *, int, int, hipStream_t);
USTD_SOLVE_INSTANTIATE(double)
USTD_SOLVE_INSTANTIATE(float)
#undef USTD_SOLVE_INSTANTIATE

hipError_t launch_residual64(const RowMap &m, int G, int u, const double *x, double *res, double *part, double *out,
                             hipStream_t st) {
    const int grid = solve_grid(m, G);
    USTD_DISPATCH_G(G, residual64_kernel<GG><<<grid, 256, 0, st>>>(m, u, x, res, part));
    reduce3_kernel<<<1, 256, 0, st>>>(part, grid, out);
    return hipGetLastError();
}

hipError_t launch_project(int n, double *x, const double *mean_src, int grid, hipStream_t st) {
    project_kernel<<<grid, 256, 0, st>>>(n, x, mean_src);
    return hipGetLastError();
}

}  // namespace ustd
