// Vector kernels of the Krylov solvers (GMRES and Lanczos): the start of a
// cycle, the Gram-Schmidt orthogonalisation of an Arnoldi step, the cycle's
// small least-squares problem, and the same for several problems at once.
//
// A solve runs about ten Arnoldi steps, each a product with H_eff and an
// orthogonalisation that waits for it, so short vectors are bound by latency:
// launches, chains of reductions, passes over the basis.  Vectors of up to
// GS_SMALL entries take one workgroup and one launch that reads the basis
// once (it was 256 threads reading it four times: bond 32, 4096 entries, up to
// eight vectors 23.8 -> 9.0 us); longer ones pass over the basis three times
// in four launches instead of four times in nine (bond 256, d 4, ten vectors
// 150 -> 95 us a step; 4.2 M entries, eight vectors 220 -> 161 us, 5.5 TB/s).
//
// Reductions are deterministic: a partition that depends on n alone, a fixed
// order within a block, and block partials summed in a fixed order.  The
// batched kernels run the same bodies, problem by problem.
#include "internal.h"
#include "wave.h"
#include "units.h"

#include <algorithm>
#include <cmath>

namespace ite {
namespace {

constexpr int RT = 256;                // threads of a reduction block
constexpr int GS_T = 1024;             // threads of the one-workgroup kernels
constexpr int GS_SMALL = 8 * GS_T;     // longest vector they take
constexpr int GS_KMAX = 64;            // basis vectors at most

__device__ inline void post_norms(const HostPost& post, double bn, double rn) {
    if (!post.flag) return;
    post.data[0] = bn;
    post.data[1] = rn;
    post_flag(post);
}

struct GsLDS {
    double part[GS_T / 64][GS_KMAX];
    double coef[GS_KMAX];
};

// Sum over the first NT threads' values (nothing of the others is read).
template <int NT>
__device__ inline double group_sum(double v, double (*part)[GS_KMAX]) {
    const int t = threadIdx.x;
    v = wave_sum(v);
    if (t < NT && (t & 63) == 0) part[t >> 6][0] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) s += part[w][0];
    __syncthreads();
    return s;
}

// Both classical Gram-Schmidt passes of one Arnoldi step in a workgroup of NT
// threads: w <- w - V (V^T w) twice (V: k1 vectors of length n,
// leading dimension ldv), the coefficients of the passes to col[0..k1) and
// col[64..64+k1), ||w|| to col[128] and, when vnext is given, vnext =
// w / ||w|| (0 for a zero norm).  Thread t owns the entries t, t + NT, ... of
// w and of the first KR basis vectors, in registers: what is left to read a
// second to fourth time are the vectors beyond (n = 4096: 8 stay).
template <int NT, int E, int KR>
__device__ inline void gs_small(const double* __restrict__ V, long ldv, int k1, double* __restrict__ w, int n,
                                double* __restrict__ col, double* __restrict__ vnext, const HostPost& post,
                                GsLDS& L) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int id = sum8_index(lane);
    // entries outside the vector are read from its last entry and kept zero
    unsigned at[E];
    bool in[E];
    double x[E], v[KR][E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        in[e] = t + NT * e < n;
        at[e] = in[e] ? t + NT * e : n - 1;
        x[e] = in[e] ? w[at[e]] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        const double* vj = V + (j < k1 ? j : 0) * ldv;
#pragma unroll
        for (int e = 0; e < E; ++e) v[j][e] = vj[at[e]];
    }
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        {
            double acc[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                acc[j] = 0.0;
                if (j < KR)
#pragma unroll
                    for (int e = 0; e < E; ++e) acc[j] += v[j % KR][e] * x[e];
            }
            const double s = sum8(acc, lane);
            if ((lane & 7) == 0 && id < KR) L.part[wv][id] = s;
        }
#pragma unroll 1
        for (int j = KR; j < k1; ++j) {
            const double* vj = V + j * ldv;
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < E; ++e) s += vj[at[e]] * x[e];
            s = wave_sum(s);
            if (lane == 0) L.part[wv][j] = s;
        }
        __syncthreads();
        if (t < k1) {
            double s = 0.0;
#pragma unroll
            for (int ww = 0; ww < NT / 64; ++ww) s += L.part[ww][t];
            L.coef[t] = s;
            col[64 * pass + t] = s;
            if (post.flag) post.data[64 * pass + t] = s;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < KR; ++j)
            if (j < k1) {
                const double c = L.coef[j];
#pragma unroll
                for (int e = 0; e < E; ++e) x[e] -= c * v[j][e];
            }
#pragma unroll 1
        for (int j = KR; j < k1; ++j) {
            const double c = L.coef[j];
            const double* vj = V + j * ldv;
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] -= c * vj[at[e]];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) x[e] = in[e] ? x[e] : 0.0;
        // (the partials of the next pass are written after this pass's last
        // read of them, the coefficients after the barrier that follows)
    }
    double ss = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) ss += x[e] * x[e];
    const double nrm = sqrt(fmax(group_sum<NT>(ss, L.part), 0.0));
    if (t == 0) {
        col[128] = nrm;
        if (post.flag) post.data[128] = nrm;
    }
    const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    if (post.flag && t == 0) post_flag(post);   // the coefficients are this wavefront's too (k1 <= 64)
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (in[e]) {
            w[at[e]] = x[e];
            if (vnext) vnext[at[e]] = x[e] * inv;
        }
}

// Threads, entries and resident basis vectors of a thread by length: four
// entries a thread where that makes at most 1024 threads (fewer wavefronts to
// sum over), eight beyond; the registers of 1024 threads hold 32 doubles of
// the basis in the first case and 16 next to the longer vector.
enum { GS_1K = 0, GS_4K = 1, GS_8K = 2, GS_LONG = 3 };
__host__ __device__ inline int gs_class(long n) {
    return n <= 1024 ? GS_1K : n <= 4096 ? GS_4K : n <= GS_SMALL ? GS_8K : GS_LONG;
}
template <int CLASS> struct GsShape;
template <> struct GsShape<GS_1K> { static constexpr int NT = 256, E = 4, KR = 8; };
template <> struct GsShape<GS_4K> { static constexpr int NT = 1024, E = 4, KR = 8; };
template <> struct GsShape<GS_8K> { static constexpr int NT = 1024, E = 8, KR = 2; };

template <int CLASS>
__global__ __launch_bounds__(GsShape<CLASS>::NT) void gs_small_kernel(const double* V, long ldv, int k1, double* w,
                                                                      int n, double* col, double* vnext,
                                                                      HostPost post) {
    typedef GsShape<CLASS> S;
    __shared__ GsLDS L;
    gs_small<S::NT, S::E, S::KR>(V, ldv, k1, w, n, col, vnext, post, L);
}

// The start of a cycle: r = b - V_0 (V_0 holds A x) or r = b, norms[0] =
// ||b||, norms[1] = ||r||, V_0 = r / ||r|| (0 for a zero norm).
template <int NT>
__device__ inline void start_small(const double* __restrict__ b, double* __restrict__ v0, bool ax, int n,
                                   double* __restrict__ norms, const HostPost& post, GsLDS& L) {
    const int t = threadIdx.x;
    double r[8];
    double bb = 0.0, rr = 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int i = t + NT * e;
        const bool in = t < NT && i < n;
        const double x = in ? b[i] : 0.0;
        r[e] = in && ax ? x - v0[i] : x;
        bb += x * x;
        rr += r[e] * r[e];
    }
    bb = group_sum<NT>(bb, L.part);
    rr = group_sum<NT>(rr, L.part);
    const double bn = sqrt(fmax(bb, 0.0)), rn = sqrt(fmax(rr, 0.0));
    if (t == 0) {
        norms[0] = bn;
        norms[1] = rn;
        post_norms(post, bn, rn);
    }
    const double inv = rn > 0.0 ? 1.0 / rn : 0.0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int i = t + NT * e;
        if (t < NT && i < n) v0[i] = r[e] * inv;
    }
}
__device__ inline void start_small_any(const double* b, double* v0, bool ax, int n, double* norms,
                                       const HostPost& post, GsLDS& L) {
    if (n <= 2048) start_small<256>(b, v0, ax, n, norms, post, L);
    else start_small<1024>(b, v0, ax, n, norms, post, L);
}
__global__ __launch_bounds__(GS_T) void start_small_kernel(const double* b, double* v0, bool ax, int n, double* norms,
                                                           double* stats, HostPost post) {
    __shared__ GsLDS L;
    if (stats && threadIdx.x < 8) stats[threadIdx.x] = 0.0;
    start_small_any(b, v0, ax, n, norms, post, L);
}

// ---------------------------------------------------------------------------
// Longer vectors: block vb of vg; partials of the first pass at part[j vg + vb],
// of the second from 16 vg on, of the norms from 32 vg on.
// ---------------------------------------------------------------------------

struct BlockLDS {
    double part[RT / 64][16];
    double coef[16];
};

// The coefficients from the blocks' partials, in every block: lane-strided
// sums in a fixed order, four wavefronts over the k1 values.
__device__ inline void sum_partials(const double* __restrict__ part, int k1, int vg, BlockLDS& L) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int j = wv; j < k1; j += RT / 64) {
        double s = 0.0;
        for (int b = lane; b < vg; b += 64) s += part[(size_t)j * vg + b];
        s = wave_sum(s);
        if (lane == 0) L.coef[j] = s;
    }
    __syncthreads();
}

// The block's sums of acc[0..k1) to part[j vg + vb].
template <int KMAX>
__device__ inline void put_partials(double (&acc)[KMAX], int k1, int vb, int vg, double* __restrict__ part,
                                    BlockLDS& L) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    __syncthreads();
#pragma unroll
    for (int j0 = 0; j0 < KMAX; j0 += 8) {
        double a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = j0 + j < KMAX ? acc[(j0 + j) % KMAX] : 0.0;
        const double s = sum8(a, lane);
        if ((lane & 7) == 0) L.part[wv][j0 + sum8_index(lane)] = s;
    }
    __syncthreads();
    if (t < k1) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < RT / 64; ++w) s += L.part[w][t];
        part[(size_t)t * vg + vb] = s;
    }
}

// PASS 0: the dot products V_j . w.  PASS 1: w -= V h1 with the first pass's
// sums, and the dot products with the new w (one read of the basis for both).
// PASS 2: w -= V h2, and w . w.
template <int KMAX, int PASS>
__device__ inline void gs_block(const double* __restrict__ V, long ldv, int k1, double* __restrict__ w, size_t n,
                                int vb, int vg, double* __restrict__ part, double* __restrict__ col, BlockLDS& L) {
    if (PASS > 0) {
        sum_partials(part + (size_t)(PASS - 1) * 16 * vg, k1, vg, L);
        if (vb == 0 && threadIdx.x < k1) col[64 * (PASS - 1) + threadIdx.x] = L.coef[threadIdx.x];
    }
    constexpr int NA = PASS == 2 ? 1 : KMAX;
    double acc[NA], c[KMAX];
#pragma unroll
    for (int j = 0; j < NA; ++j) acc[j] = 0.0;
#pragma unroll
    for (int j = 0; j < KMAX; ++j) c[j] = PASS > 0 && j < k1 ? L.coef[j] : 0.0;
    const size_t stride = (size_t)vg * RT;
    for (size_t i = (size_t)vb * RT + threadIdx.x; i < n; i += stride) {
        double x = w[i];
        double v[KMAX];
#pragma unroll
        for (int j = 0; j < KMAX; ++j) v[j] = j < k1 ? V[(size_t)j * ldv + i] : 0.0;
        if (PASS > 0) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < KMAX; ++j) s += c[j] * v[j];
            x -= s;
            w[i] = x;
        }
        if (PASS == 2) acc[0] += x * x;
        else {
#pragma unroll
            for (int j = 0; j < NA; ++j) acc[j] += v[j] * x;
        }
    }
    put_partials<NA>(acc, PASS == 2 ? 1 : k1, vb, vg, part + (size_t)PASS * 16 * vg, L);
}

template <int KMAX, int PASS>
__global__ __launch_bounds__(RT) void gs_kernel(const double* __restrict__ V, long ldv, int k1, double* __restrict__ w,
                                                size_t n, double* __restrict__ part, double* __restrict__ col) {
    __shared__ BlockLDS L;
    gs_block<KMAX, PASS>(V, ldv, k1, w, n, blockIdx.x, gridDim.x, part, col, L);
}

// vnext = w / ||w|| and the norm itself, from the blocks' partials.
__device__ inline void scale_block(const double* __restrict__ w, size_t n, int vb, int vg,
                                   const double* __restrict__ part, double* __restrict__ col, int k1,
                                   double* __restrict__ vnext, const HostPost& post, BlockLDS& L) {
    sum_partials(part, 1, vg, L);
    const double nrm = sqrt(fmax(L.coef[0], 0.0));
    if (vb == 0 && threadIdx.x < 64) {
        const int t = threadIdx.x;
        if (t == 0) col[128] = nrm;
        if (post.flag) {
            if (t < k1) {
                post.data[t] = col[t];
                post.data[64 + t] = col[64 + t];
            }
            if (t == 0) {
                post.data[128] = nrm;
                post_flag(post);
            }
        }
    }
    if (!vnext) return;
    const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    for (size_t i = (size_t)vb * RT + threadIdx.x; i < n; i += (size_t)vg * RT) vnext[i] = w[i] * inv;
}
__global__ __launch_bounds__(RT) void gs_scale_kernel(const double* __restrict__ w, size_t n, int vg,
                                                      const double* __restrict__ part, double* __restrict__ col,
                                                      int k1, double* __restrict__ vnext, HostPost post) {
    __shared__ BlockLDS L;
    scale_block(w, n, blockIdx.x, vg, part + (size_t)32 * vg, col, k1, vnext, post, L);
}

__device__ inline void start_block(const double* __restrict__ b, double* __restrict__ v0, bool ax, size_t n, int vb,
                                   int vg, double* __restrict__ part, BlockLDS& L) {
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (size_t i = (size_t)vb * RT + threadIdx.x; i < n; i += (size_t)vg * RT) {
        const double x = b[i];
        const double r = ax ? x - v0[i] : x;
        v0[i] = r;
        acc[0] += x * x;
        acc[1] += r * r;
    }
    put_partials<8>(acc, 2, vb, vg, part, L);
}
__device__ inline void start_scale_block(double* __restrict__ v0, size_t n, int vb, int vg,
                                         const double* __restrict__ part, double* __restrict__ norms,
                                         const HostPost& post, BlockLDS& L) {
    sum_partials(part, 2, vg, L);
    const double bn = sqrt(fmax(L.coef[0], 0.0)), rn = sqrt(fmax(L.coef[1], 0.0));
    if (vb == 0 && threadIdx.x == 0) {
        norms[0] = bn;
        norms[1] = rn;
        post_norms(post, bn, rn);
    }
    const double inv = rn > 0.0 ? 1.0 / rn : 0.0;
    for (size_t i = (size_t)vb * RT + threadIdx.x; i < n; i += (size_t)vg * RT) v0[i] *= inv;
}
__global__ __launch_bounds__(RT) void start_kernel(const double* __restrict__ b, double* __restrict__ v0, bool ax,
                                                   size_t n, double* __restrict__ part, double* __restrict__ stats) {
    __shared__ BlockLDS L;
    if (stats && blockIdx.x == 0 && threadIdx.x < 8) stats[threadIdx.x] = 0.0;
    start_block(b, v0, ax, n, blockIdx.x, gridDim.x, part, L);
}
__global__ __launch_bounds__(RT) void start_scale_kernel(double* __restrict__ v0, size_t n,
                                                         const double* __restrict__ part, double* __restrict__ norms,
                                                         HostPost post) {
    __shared__ BlockLDS L;
    start_scale_block(v0, n, blockIdx.x, gridDim.x, part, norms, post, L);
}

// ---------------------------------------------------------------------------
// Least squares of a cycle
// ---------------------------------------------------------------------------

// The small least-squares problem of one GMRES cycle in one wavefront, lane k
// holding column k of the Hessenberg matrix: the columns of the cycle's
// Arnoldi steps are hd[k * HESS_HC + i] (first Gram-Schmidt pass), + 64
// (second pass), + 128 (the norm of the next vector); norms: ||b|| and
// beta = ||r0||.  Givens rotation i comes from
// column i and is applied to all later columns at once (they would wait for
// it one by one otherwise: 16.5 us a cycle of ten, now 6.5), and the residual
// estimate |g_(k+1)| is tracked; an Arnoldi step whose next norm is <= 1e-14
// beta ends the cycle (invariant subspace); y solves R y = g by back
// substitution, column by column (zero beyond the steps used).  stats (per
// local solve, zeroed before the first cycle): [0] relative residual
// estimate, [1] products whose results enter the solution, [2] ITE_FLAG_*
// bits, [3] 1 once a cycle found an invariant subspace or a zero residual
// (later cycles then change nothing), [4] the residual products alone.
// Hs: LDS of R, rows padded so that a row's lanes and a column's spread over
// the banks.
constexpr int HESS_LD = HESS_KMAX + 1;
__device__ void hess_solve_one(const double* __restrict__ hd, const double* __restrict__ norms, int mm, double* __restrict__ y,
                               double* __restrict__ stats, int r_product, int last_cycle,
                               double (*Hs)[HESS_LD]) {
    const int k = threadIdx.x;
    if (stats[3] != 0.0) {
        if (k < mm) y[k] = 0.0;
        return;
    }
    double products = stats[1] + (r_product ? 1.0 : 0.0);
    const double rproducts = stats[4] + (r_product ? 1.0 : 0.0);   // FP64 even when the others are not
    const int flags0 = (int)stats[2];
    const double bnorm = norms[0], beta = norms[1];
    if (!(beta > 0.0)) {
        if (k < mm) y[k] = 0.0;
        if (k == 0) {
            stats[0] = bnorm > 0.0 ? beta / bnorm : 0.0;
            stats[1] = products;
            stats[3] = 1.0;
            stats[4] = rproducts;
        }
        return;
    }
    const double* col = hd + (size_t)min(k, mm - 1) * HESS_HC;
    const double hnext = col[128];
    for (int i = 0; i < mm; ++i) {
        const double h = i <= k ? col[i] + col[64 + i] : 0.0;
        if (k < mm) Hs[i][k] = h;
    }
    __syncthreads();
    double cur = k < mm ? Hs[0][k] : 0.0;   // H[i][k] after the rotations before i
    double g = 0.0, gi = beta;              // this lane's g and the running one
    double diag = 0.0;
    int kused = mm;
    bool breakdown = false;
    for (int i = 0; i < mm; ++i) {
        const double next = i + 1 < mm && k < mm ? Hs[i + 1][k] : 0.0;
        const double a = lane_value(cur, i), b = lane_value(hnext, i);
        const double rr = hypot(a, b);
        const double cs = rr > 0.0 ? a / rr : 1.0, sn = rr > 0.0 ? b / rr : 0.0;
        if (k == i) {
            diag = rr;
            g = cs * gi;
        }
        gi = -sn * gi;
        if (k > i && k < mm) Hs[i][k] = cs * cur + sn * next;
        cur = -sn * cur + cs * next;
        if (b <= 1e-14 * beta) {
            kused = i + 1;
            breakdown = true;
            break;
        }
    }
    __syncthreads();
    double mine = 0.0;
    for (int j = kused - 1; j >= 0; --j) {
        const double dgn = lane_value(diag, j);
        const double yj = dgn != 0.0 ? lane_value(g, j) / dgn : 0.0;
        if (k == j) mine = yj;
        if (k < j) g -= Hs[k][j] * yj;
    }
    if (k < mm) y[k] = mine;
    if (k == 0) {
        int flags = flags0;
        if (breakdown) {
            flags |= ITE_FLAG_BREAKDOWN;
            stats[3] = 1.0;
        } else if (last_cycle) {
            flags |= ITE_FLAG_BUDGET_EXHAUSTED;
        }
        stats[0] = bnorm > 0.0 ? fabs(gi) / bnorm : 0.0;
        stats[1] = products + kused;
        stats[2] = (double)flags;
        stats[4] = rproducts;
    }
}

__global__ __launch_bounds__(64) void hess_solve_kernel(const double* __restrict__ hd, const double* __restrict__ norms,
                                                        int mm, double* __restrict__ y, double* __restrict__ stats,
                                                        int r_product, int last_cycle) {
    __shared__ double Hs[HESS_KMAX][HESS_LD];
    hess_solve_one(hd, norms, mm, y, stats, r_product, last_cycle, Hs);
}

// ---------------------------------------------------------------------------
// Batched
// ---------------------------------------------------------------------------

template <int CLASS>
__global__ __launch_bounds__(GsShape<CLASS>::NT) void batch_gs_small_kernel(const BatchVec* __restrict__ d, int G,
                                                                            int k, int mm) {
    typedef GsShape<CLASS> S;
    __shared__ GsLDS L;
    for (int g = blockIdx.x; g < G; g += gridDim.x) {
        const BatchVec& p = d[g];
        if (gs_class(p.n) != CLASS) continue;
        double* vnext = k + 1 < mm ? p.V + (size_t)(k + 1) * p.n : nullptr;
        gs_small<S::NT, S::E, S::KR>(p.V, p.n, k + 1, p.w, (int)p.n, p.hd + (size_t)k * HESS_HC, vnext,
                                     HostPost{}, L);
        __syncthreads();
    }
}

__global__ __launch_bounds__(GS_T) void batch_start_small_kernel(const BatchVec* __restrict__ d, int G, int mm,
                                                                 int first) {
    __shared__ GsLDS L;
    for (int g = blockIdx.x; g < G; g += gridDim.x) {
        const BatchVec& p = d[g];
        if (gs_class(p.n) == GS_LONG) continue;
        if (first && threadIdx.x < 8) p.stats[threadIdx.x] = 0.0;
        start_small_any(p.b, p.V, true, (int)p.n, p.hd + (size_t)mm * HESS_HC, HostPost{}, L);
        __syncthreads();
    }
}

// Block units of the long problems: PASS 0..2 of gs_block, 3 the scaling,
// 4 and 5 the start of a cycle.
template <int KMAX, int PASS>
__global__ __launch_bounds__(RT) void batch_gs_kernel(const BatchVec* __restrict__ d, int G,
                                                      const int* __restrict__ tot, int k, int mm, int first) {
    __shared__ BlockLDS L;
    const int total = tot[BT_RED];
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int g = unit_problem(u, G, [&](int q) { return d[q].red_start; });
        const BatchVec& p = d[g];
        const int vb = u - p.red_start;
        if (gs_class(p.n) != GS_LONG || vb >= p.nb) continue;
        double* col = p.hd + (size_t)k * HESS_HC;
        if constexpr (PASS < 3) {
            gs_block<KMAX, PASS>(p.V, p.n, k + 1, p.w, p.n, vb, p.nb, p.part, col, L);
        } else if constexpr (PASS == 3) {
            scale_block(p.w, p.n, vb, p.nb, p.part + (size_t)32 * p.nb, col, k + 1,
                        k + 1 < mm ? p.V + (size_t)(k + 1) * p.n : nullptr, HostPost{}, L);
        } else if constexpr (PASS == 4) {
            if (first && vb == 0 && threadIdx.x < 8) p.stats[threadIdx.x] = 0.0;
            start_block(p.b, p.V, true, p.n, vb, p.nb, p.part, L);
        } else {
            start_scale_block(p.V, p.n, vb, p.nb, p.part, p.hd + (size_t)mm * HESS_HC, HostPost{}, L);
        }
        __syncthreads();   // the LDS is the next unit's
    }
}

__global__ __launch_bounds__(64) void batch_hess_kernel(const BatchVec* __restrict__ d, int G, int mm, int r_product,
                                                        int last_cycle) {
    __shared__ double Hs[HESS_KMAX][HESS_LD];
    for (int g = blockIdx.x; g < G; g += gridDim.x) {
        const BatchVec& p = d[g];
        hess_solve_one(p.hd, p.hd + (size_t)mm * HESS_HC, mm, p.y, p.stats, r_product, last_cycle, Hs);
        __syncthreads();
    }
}

}  // namespace

int krylov_class(size_t n) { return gs_class((long)n); }

void krylov_start(const double* b, double* v0, bool ax, size_t n, double* norms, double* part, double* stats,
                  hipStream_t s, HostPost post) {
    if (n == 0) return;
    if (gs_class((long)n) != GS_LONG) {
        hipLaunchKernelGGL(start_small_kernel, dim3(1), dim3(n <= 2048 ? 256 : GS_T), 0, s, b, v0, ax, (int)n, norms,
                           stats, post);
    } else {
        const dim3 grid(reduce_blocks(n));
        hipLaunchKernelGGL(start_kernel, grid, dim3(RT), 0, s, b, v0, ax, n, part, stats);
        hipLaunchKernelGGL(start_scale_kernel, grid, dim3(RT), 0, s, v0, n, part, norms, post);
    }
    HIP_CHECK(hipGetLastError());
}

// part[j nb + b]: block b's share of V_j . w for j < k1 <= 16.  The kernel fetches
// all of an entry's values before it uses one (2.4 M entries, 16 vectors: 52 us, 40 by the vectors alone at 8 TB/s;
// 117 with each product behind its own test of j).
static void gs_dots(const double* V, long ldv, int k1, double* w, size_t n, double* part, hipStream_t s) {
    const dim3 grid(reduce_blocks(n));
    if (k1 <= 4) hipLaunchKernelGGL((gs_kernel<4, 0>), grid, dim3(RT), 0, s, V, ldv, k1, w, n, part, nullptr);
    else if (k1 <= 8) hipLaunchKernelGGL((gs_kernel<8, 0>), grid, dim3(RT), 0, s, V, ldv, k1, w, n, part, nullptr);
    else hipLaunchKernelGGL((gs_kernel<16, 0>), grid, dim3(RT), 0, s, V, ldv, k1, w, n, part, nullptr);
}

template <int KMAX>
static void gs_launch(const double* V, long ldv, int k1, double* w, size_t n, double* col, double* part,
                      hipStream_t s) {
    const dim3 grid(reduce_blocks(n));
    hipLaunchKernelGGL((gs_kernel<KMAX, 0>), grid, dim3(RT), 0, s, V, ldv, k1, w, n, part, col);
    hipLaunchKernelGGL((gs_kernel<KMAX, 1>), grid, dim3(RT), 0, s, V, ldv, k1, w, n, part, col);
    hipLaunchKernelGGL((gs_kernel<KMAX, 2>), grid, dim3(RT), 0, s, V, ldv, k1, w, n, part, col);
}

void gram_schmidt(const double* V, long ldv, int k1, double* w, size_t n, double* col, double* vnext, double* part,
                  hipStream_t s, HostPost post) {
    if (n == 0) return;
    if (k1 < 1 || k1 > GS_KMAX) ITE_FAIL(ITE_EINVAL, "gram_schmidt: basis outside 1..64 vectors");
    const int cls = gs_class((long)n);
    if (cls != GS_LONG) {
#define ITE_GS(C) \
    hipLaunchKernelGGL((gs_small_kernel<C>), dim3(1), dim3(GsShape<C>::NT), 0, s, V, ldv, k1, w, (int)n, col, vnext, post)
        if (cls == GS_1K) ITE_GS(GS_1K);
        else if (cls == GS_4K) ITE_GS(GS_4K);
        else ITE_GS(GS_8K);
#undef ITE_GS
        HIP_CHECK(hipGetLastError());
        return;
    }
    const int nb = reduce_blocks(n);
    if (k1 <= 16) {
        if (k1 <= 4) gs_launch<4>(V, ldv, k1, w, n, col, part, s);
        else if (k1 <= 8) gs_launch<8>(V, ldv, k1, w, n, col, part, s);
        else gs_launch<16>(V, ldv, k1, w, n, col, part, s);
        hipLaunchKernelGGL(gs_scale_kernel, dim3(vnext ? nb : 1), dim3(RT), 0, s, w, n, nb, part, col, k1, vnext, post);
        HIP_CHECK(hipGetLastError());
        return;
    }
    // wider bases do not fit a thread's registers: separate products and
    // updates, 16 vectors at a time
    for (int pass = 0; pass < 2; ++pass) {
        for (int j0 = 0; j0 < k1; j0 += 16)
            gs_dots(V + (size_t)j0 * ldv, ldv, std::min(k1 - j0, 16), w, n, part + (size_t)j0 * nb, s);
        finish_partials(part, k1, nb, col + 64 * pass, 0, s);
        gemv_sub(V, ldv, k1, col + 64 * pass, w, n, s);
    }
    dot_partials(w, w, n, part + (size_t)32 * nb, s);
    hipLaunchKernelGGL(gs_scale_kernel, dim3(vnext ? nb : 1), dim3(RT), 0, s, w, n, nb, part, col, k1, vnext, post);
    HIP_CHECK(hipGetLastError());
}

void hess_solve(const double* hd, const double* norms, int mm, double* y, double* stats, bool r_product, bool last_cycle, hipStream_t s) {
    if (mm < 1 || mm > HESS_KMAX) ITE_FAIL(ITE_EINVAL, "hess_solve: Krylov dimension outside 1..64");
    hipLaunchKernelGGL(hess_solve_kernel, dim3(1), dim3(64), 0, s, hd, norms, mm, y, stats, (int)r_product,
                       (int)last_cycle);
    HIP_CHECK(hipGetLastError());
}

void batch_start(const BatchVec* d, int G, const int* tot, unsigned classes, int mm, bool first, hipStream_t s) {
    if (G <= 0) return;
    if (classes & ~(1u << GS_LONG))
        hipLaunchKernelGGL(batch_start_small_kernel, dim3(std::min(G, BATCH_GRID)), dim3(GS_T), 0, s, d, G, mm,
                           (int)first);
    if (classes & 1u << GS_LONG) {
        hipLaunchKernelGGL((batch_gs_kernel<4, 4>), dim3(BATCH_GRID), dim3(RT), 0, s, d, G, tot, 0, mm, (int)first);
        hipLaunchKernelGGL((batch_gs_kernel<4, 5>), dim3(BATCH_GRID), dim3(RT), 0, s, d, G, tot, 0, mm, 0);
    }
    HIP_CHECK(hipGetLastError());
}

template <int KMAX>
static void batch_gs_launch(const BatchVec* d, int G, const int* tot, int k, int mm, hipStream_t s) {
    hipLaunchKernelGGL((batch_gs_kernel<KMAX, 0>), dim3(BATCH_GRID), dim3(RT), 0, s, d, G, tot, k, mm, 0);
    hipLaunchKernelGGL((batch_gs_kernel<KMAX, 1>), dim3(BATCH_GRID), dim3(RT), 0, s, d, G, tot, k, mm, 0);
    hipLaunchKernelGGL((batch_gs_kernel<KMAX, 2>), dim3(BATCH_GRID), dim3(RT), 0, s, d, G, tot, k, mm, 0);
}

void batch_gram_schmidt(const BatchVec* d, int G, const int* tot, unsigned classes, int k, int mm,
                        hipStream_t s) {
    if (G <= 0) return;
    if (k < 0 || k >= 16) ITE_FAIL(ITE_EINVAL, "batch_gram_schmidt: at most 16 basis vectors");
    const dim3 grid(std::min(G, BATCH_GRID));
#define ITE_GS(C)            \
    if (classes & 1u << C)   \
    hipLaunchKernelGGL((batch_gs_small_kernel<C>), grid, dim3(GsShape<C>::NT), 0, s, d, G, k, mm)
    ITE_GS(GS_1K);
    ITE_GS(GS_4K);
    ITE_GS(GS_8K);
#undef ITE_GS
    if (classes & 1u << GS_LONG) {
        if (k < 4) batch_gs_launch<4>(d, G, tot, k, mm, s);
        else if (k < 8) batch_gs_launch<8>(d, G, tot, k, mm, s);
        else batch_gs_launch<16>(d, G, tot, k, mm, s);
        hipLaunchKernelGGL((batch_gs_kernel<4, 3>), dim3(BATCH_GRID), dim3(RT), 0, s, d, G, tot, k, mm, 0);
    }
    HIP_CHECK(hipGetLastError());
}

void batch_hess(const BatchVec* d, int G, int mm, bool r_product, bool last_cycle, hipStream_t s) {
    if (G <= 0) return;
    if (mm < 1 || mm > HESS_KMAX) ITE_FAIL(ITE_EINVAL, "batch_hess: Krylov dimension outside 1..64");
    hipLaunchKernelGGL(batch_hess_kernel, dim3(std::min(G, BATCH_GRID)), dim3(64), 0, s, d, G, mm, (int)r_product,
                       (int)last_cycle);
    HIP_CHECK(hipGetLastError());
}

}  // namespace ite
