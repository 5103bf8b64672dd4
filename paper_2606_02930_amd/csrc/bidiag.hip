// Householder bidiagonalisation of a two-site block and the way back from
// the singular vectors of the bidiagonal matrix to those of the block.
//
// A (P x N, P >= N, row-major) becomes B = Q^T A Z, upper bidiagonal (Golub
// and Kahan): in step c a reflector on the rows from c on clears column c
// below the diagonal, one on the columns from c + 1 on clears row c right of
// the superdiagonal.  While more than 192 rows are left a step is one pass over
// the trailing block (bd_step_kernel: both reflectors applied to a row while its
// entries are in registers, and its share of the next step's column
// products taken) and one sum over the workgroups (bd_sum_kernel), or both in
// one launch from 512 rows and columns on (bd_step1_kernel); the rest is
// done by one workgroup in its registers (bd_tail_kernel).  Bound by the
// latency of a step: 5 to 7 us at 200 to 512 columns,
// 14 us at 2048 (38 MB read and written by it on average there), 1.2 to 2 us
// inside one workgroup.  Two launches a step that each read and wrote the
// block (columns, then rows) took 9 us and 31 us.
//
// The reflectors are kept as rows of VQ and VP (zero before the first entry,
// which is one), both sizes padded with zeros to multiples of 16.  bd_vectors applies them in blocks of 16 in the
// compact WY form (Schreiber and Van Loan) to the kept singular vectors: a
// workgroup holds 16 vectors in the accumulator registers of its wavefronts
// for all blocks, since the FP64 MFMA accumulator layout (element r of lane
// group g = row 4 r + g) is the B operand layout of K step r.
#include "internal.h"
#include "wave.h"

#include <algorithm>

namespace ite {
namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));

constexpr int WYB = 16;      // reflectors per block
__host__ __device__ inline int pad16(int n) { return (n + 15) & ~15; }

// The reflector of x[0..len) (LAPACK's convention: beta = -sign(alpha) ||x||,
// tau = (beta - alpha) / beta, v = x / (alpha - beta) with v_0 = 1; tau = 0
// when x_1.. = 0) from alpha = x_0 and sg = x_1^2 + ...  Below ||x|| = 1e-140 the
// squares lose digits or vanish, and a reflector formed from them would not be
// orthogonal: such an x counts as zero (split scales blocks that are that small
// altogether).
struct Refl {
    double beta, tau, scale;
};
__device__ inline Refl reflector(double alpha, double sg) {
    Refl r{alpha, 0.0, 0.0};
    const double s2 = alpha * alpha + sg;
    if (sg > 0.0 && s2 > 1e-280) {
        if (s2 < 1e280) {
            // the two reciprocals side by side instead of a square root and
            // two divisions in a chain
            const double y = recip_sqrt(s2), nrm = s2 * y;
            r.beta = alpha >= 0.0 ? -nrm : nrm;
            r.tau = 1.0 + fabs(alpha) * y;
            r.scale = recip(alpha - r.beta);
        } else {
            const double nrm = sqrt(s2);
            r.beta = alpha >= 0.0 ? -nrm : nrm;
            r.tau = (r.beta - alpha) / r.beta;
            r.scale = 1.0 / (alpha - r.beta);
        }
    } else if (!(sg >= 0.0)) {
        r.beta = r.tau = sg;     // NaN stays NaN (dc_leaf_kernel looks for it)
    }
    return r;
}
// The part of a row entry r that the left reflector takes away (p: the product
// of its column with the pivot column), and what it leaves.  Rounded the same way
// wherever they are formed: of a row that is almost finished only rounding is
// left, and the reflector that is applied has to be the one that is kept.
__device__ inline double left_part(const Refl& h, double r, double p) {
#pragma clang fp contract(off)
    const double sp = h.scale * p;
    return h.tau * (r + sp);
}
__device__ inline double left_rest(double r, double z) {
#pragma clang fp contract(off)
    return r - z;
}
// The rows past the last reflector of either side.
__device__ inline void clear_padding(int P, int N, double* VQ, double* VP, long id, long all) {
    for (long i = (long)N * pad16(P) + id; i < (long)pad16(N) * pad16(P); i += all) VQ[i] = 0.0;
    for (long i = (long)(N - 1) * pad16(N) + id; i < (long)pad16(N) * pad16(N); i += all) VP[i] = 0.0;
}

// A <- theta (P x N), or theta^T when tr (theta then N x P).
__global__ __launch_bounds__(256) void bd_load_kernel(const double* __restrict__ theta, int P, int N, int tr,
                                                      double* __restrict__ A, double* __restrict__ VQ,
                                                      double* __restrict__ VP) {
    __shared__ double tile[32][33];
    clear_padding(P, N, VQ, VP, ((long)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x,
                  (long)gridDim.x * gridDim.y * 256);
    const int x = threadIdx.x & 31, y0 = threadIdx.x >> 5;
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;      // of A
    if (tr) {
        for (int y = y0; y < 32; y += 8)
            if (c0 + y < N && r0 + x < P) tile[x][y] = theta[(long)(c0 + y) * P + r0 + x];
        __syncthreads();
    }
    for (int y = y0; y < 32; y += 8) {
        const int r = r0 + y, c = c0 + x;
        if (r >= P || c >= N) continue;
        A[(long)r * N + c] = tr ? tile[y][x] : theta[(long)r * N + c];
    }
}

// Step c in one pass over the rows below it.  p[j] = sum_(i > c) A[i][c] A[i][j]
// (j >= c) is all that is needed from the other rows: with it every workgroup has
// the left reflector and the updated row c, and from that the right reflector.
// Each row takes both reflectors, and its share of the next step's p follows
// while it is in registers: part[workgroup][j], summed by bd_sum_kernel.  start:
// no step, only the products for the first column (c = -1).
//
// A thread has Q columns of all the workgroup's rows, so its parts of row c, of
// the reflectors and of the products stay in its registers, and what crosses
// wavefronts is a norm and a number a row.  (With a wavefront a row the
// reflectors were read from LDS by every row and the products summed through it:
// 13.2 us a step over 2048 to 1024 columns, now 11.0; 7.4 over 1024 to 512, now
// 6.5.)
constexpr int BS_NW = 8;            // rows and wavefronts of a workgroup
constexpr int BS_NT = 64 * BS_NW;
template <int Q>
__global__ __launch_bounds__(BS_NT) void bd_step_kernel(BdWork b, int c, bool start) {
    constexpr int R = BS_NW;
    __shared__ double sh[BS_NW], dots[BS_NW][R];
    const int P = b.P, N = b.N, c1 = c + 1, len = N - c1;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    // a row has the same workgroup number in every step; the first ones finish
    const int blk0 = c1 / R, i0 = blockIdx.x * R;
    if ((int)blockIdx.x < blk0) return;
    // row c and the products are needed first, so they are asked for first; the
    // rows arrive while the reflectors are formed
    const double* rowc = b.A + (long)max(c, 0) * N;
    double rc[Q], pc[Q], a[R][Q];
    double alpha = 0.0, sg = 0.0, first = 0.0, pfirst = 0.0;
    if (!start) {
        alpha = rowc[c];
        sg = b.p[c];
        if (len > 0) {
            first = rowc[c1];
            pfirst = b.p[c1];
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int j = t + BS_NT * q;
            rc[q] = j < len ? rowc[c1 + j] : 0.0;
            pc[q] = j < len ? b.p[c1 + j] : 0.0;
        }
    }
    // lane r: the entries of row i0 + r in columns c and c + 1
    double xl = 0.0, xnl = 0.0;
    const int il = i0 + (lane & (R - 1));
    if (il >= c1 && il < P) {
        if (!start) xl = b.A[(long)il * N + c];
        if (len > 0) xnl = b.A[(long)il * N + c1];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = i0 + r;
        const double* Ai = b.A + (long)i * N + c1;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int j = t + BS_NT * q;
            a[r][q] = i >= c1 && i < P && j < len ? Ai[j] : 0.0;
        }
    }
    if (!start) {
        const Refl h = reflector(alpha, sg);
        double z[Q], u[Q], n2 = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            z[q] = left_part(h, rc[q], pc[q]);
            u[q] = left_rest(rc[q], z[q]);
            if (t + BS_NT * q > 0) n2 += u[q] * u[q];
        }
        n2 = wave_sum(n2);
        if (lane == 0) sh[w] = n2;
        __syncthreads();
        n2 = sh[0];
#pragma unroll
        for (int q = 1; q < BS_NW; ++q) n2 += sh[q];
        const double z0 = left_part(h, first, pfirst);
        const Refl k = reflector(len > 0 ? left_rest(first, z0) : 0.0, n2);
#pragma unroll
        for (int q = 0; q < Q; ++q) u[q] = t + BS_NT * q == 0 ? 1.0 : u[q] * k.scale;
        const int ldq = pad16(P), ldp = pad16(N);
        if ((int)blockIdx.x == blk0) {
            double* vq = b.VQ + (long)c * ldq;
            for (int q = t; q <= c; q += BS_NT) vq[q] = q == c ? 1.0 : 0.0;
            for (int q = P + t; q < ldq; q += BS_NT) vq[q] = 0.0;
            if (len > 0) {
                double* vp = b.VP + (long)c * ldp;
                for (int q = t; q < c1; q += BS_NT) vp[q] = 0.0;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (c1 + t + BS_NT * q < N) vp[c1 + t + BS_NT * q] = u[q];
                for (int q = N + t; q < ldp; q += BS_NT) vp[q] = 0.0;
            }
            if (t == 0) {
                b.tauq[c] = h.tau;
                b.d[c] = h.beta;
                b.taup[c] = k.tau;
                b.e[c] = k.beta;
            }
        }
        const double vl = xl * h.scale;
        if (t < R && il >= c1 && il < P) b.VQ[(long)c * ldq + il] = vl;
        double v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = lane_value(vl, r);
        if (len == 0) return;
        double d[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            d[r] = 0.0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                a[r][q] -= v[r] * z[q];
                d[r] += a[r][q] * u[q];
            }
        }
        const double mine = sum8(d, lane);
        if ((lane & 7) == 0) dots[w][sum8_index(lane)] = mine;
        __syncthreads();
        // lane 8 s + r: wavefront s's part of row r
        double dr = dots[lane >> 3][lane & 7];
        dr += dpp_move<0x128, 0xf>(dr);                 // row_ror:8
        dr = swap_add16(dr, dr);
        dr = k.tau * swap_add32(dr, dr);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double e = lane_value(dr, r);
            const int i = i0 + r;
            const bool in = i >= c1 && i < P;
            double* Ai = b.A + (long)i * N + c1;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                a[r][q] -= e * u[q];
                if (in && t + BS_NT * q < len) Ai[t + BS_NT * q] = a[r][q];
            }
        }
        xnl = xnl - vl * z0 - dr;
    }
    // the next step's column products: rows below its own row
    if (il <= c1 || il >= P) xnl = 0.0;
    double xn[R];
#pragma unroll
    for (int r = 0; r < R; ++r) xn[r] = lane_value(xnl, r);
    double* part = b.part + (long)blockIdx.x * N + c1;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) s += xn[r] * a[r][q];
        if (t + BS_NT * q < len) part[t + BS_NT * q] = s;
    }
}

// The same for rows of any length, in memory, with z and u formed again where they
// are used; a wavefront a row.  A row is read three times and written once: 2100 rows
// and columns take 29 ms in all (2048: 24), 2600 61, 3200 107, 4096 200 (the Jacobi
// before: 107, 146, 232, 445, and 265 to 1017 for a graded block).
constexpr int BS_CH = 512;          // columns of a row of products in LDS
__global__ __launch_bounds__(BS_NT) void bd_step_long_kernel(BdWork b, int c, bool start) {
    constexpr int NT = BS_NT;
    __shared__ double buf[BS_NW][BS_CH];
    __shared__ double sh[BS_NW];
    const int P = b.P, N = b.N, c1 = c + 1, len = N - c1;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int blk0 = c1 / BS_NW, i = blockIdx.x * BS_NW + w;
    if ((int)blockIdx.x < blk0) return;
    const bool in = i >= c1 && i < P;
    double* Ai = b.A + (long)i * N + c1;
    const double* rowc = b.A + (long)max(c, 0) * N;
    double xn;       // the row's entry in the next step's column
    if (!start) {
        const double x = in ? Ai[-1] : 0.0;
        const Refl h = reflector(rowc[c], b.p[c]);
        auto left = [&](int j) { return left_part(h, rowc[c1 + j], b.p[c1 + j]); };
        double n2 = 0.0;
        for (int j = 1 + t; j < len; j += NT) {
            const double r = left_rest(rowc[c1 + j], left(j));
            n2 += r * r;
        }
        n2 = wave_sum(n2);
        if (lane == 0) sh[w] = n2;
        __syncthreads();
        n2 = sh[0];
#pragma unroll
        for (int q = 1; q < BS_NW; ++q) n2 += sh[q];
        const Refl k = reflector(len > 0 ? left_rest(rowc[c1], left(0)) : 0.0, n2);
        auto uat = [&](int j) { return j == 0 ? 1.0 : left_rest(rowc[c1 + j], left(j)) * k.scale; };
        const int ldq = pad16(P), ldp = pad16(N);
        if ((int)blockIdx.x == blk0) {
            double* vq = b.VQ + (long)c * ldq;
            for (int q = t; q <= c; q += NT) vq[q] = q == c ? 1.0 : 0.0;
            for (int q = P + t; q < ldq; q += NT) vq[q] = 0.0;
            if (len > 0) {
                double* vp = b.VP + (long)c * ldp;
                for (int q = t; q < ldp; q += NT) vp[q] = q < c1 || q >= N ? 0.0 : uat(q - c1);
            }
            if (t == 0) {
                b.tauq[c] = h.tau;
                b.d[c] = h.beta;
                b.taup[c] = k.tau;
                b.e[c] = k.beta;
            }
        }
        const double v = x * h.scale;
        if (in && lane == 0) b.VQ[(long)c * ldq + i] = v;
        if (len == 0) return;
        double d = 0.0;
        for (int j = lane; in && j < len; j += 64) d += (Ai[j] - v * left(j)) * uat(j);
        d = k.tau * wave_sum(d);
        double head = 0.0;
        for (int j = lane; in && j < len; j += 64) {
            const double r = Ai[j] - v * left(j) - d * uat(j);
            Ai[j] = r;
            if (j == 0) head = r;
        }
        xn = lane_value(head, 0);
    } else {
        xn = in ? Ai[0] : 0.0;
    }
    // the next step's column products: rows below its own row
    if (i == c1 || !in) xn = 0.0;
    double* part = b.part + (long)blockIdx.x * N + c1;
    for (int c0 = 0; c0 < len; c0 += BS_CH) {
        if (c0 > 0) __syncthreads();
        for (int j = lane; j < BS_CH; j += 64) buf[w][j] = (in && c0 + j < len) ? xn * Ai[c0 + j] : 0.0;
        __syncthreads();
        for (int j = t; j < BS_CH && c0 + j < len; j += NT) {
            double s = buf[0][j];
#pragma unroll
            for (int q = 1; q < BS_NW; ++q) s += buf[q][j];
            part[c0 + j] = s;
        }
    }
}

// p[j] = the sum over the products of workgroups q0 .. np - 1, j >= c.
__global__ __launch_bounds__(1024) void bd_sum_kernel(BdWork b, int c, int q0, int np) {
    __shared__ double sh[16][17];
    const int N = b.N, t = threadIdx.x, tx = t & 15, ty = t >> 4, j = c + blockIdx.x * 16 + tx;
    double s = 0.0;
    if (j < N)
        for (int q = q0 + ty; q < np; q += 64) s += b.part[(long)q * N + j];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if ((ty & 3) == 0) sh[t >> 6][tx] = s;
    __syncthreads();
    if (t < 16 && j < N) {
        s = sh[0][tx];
#pragma unroll
        for (int q = 1; q < 16; ++q) s += sh[q][tx];
        b.p[j] = s;
    }
}

// The same step in one launch, for up to 64 CPL columns from c on and few
// workgroups: NW wavefronts of R rows each, so that every workgroup can sum
// the products of all (src, workgroups q0 .. ns - 1) by itself.  That sum is
// all loads in flight at once; it and the redundant reflectors grow with the
// rows a workgroup has less, the row work with those it has more: 8
// wavefronts of 2 rows take 5.1 us at 256 rows and columns and 6.7 at 512
// (8 x 1: 5.4 and 7.2, 8 x 4: 6.1 and 8.1, 16 x 2: 6.9 and 8.7; step and sum as
// two launches 7.1 and 8.0).
template <int CPL, int R, int NW>
__global__ __launch_bounds__(64 * NW) void bd_step1_kernel(BdWork b, int c, const double* __restrict__ src, int q0, int ns,
                                                        double* __restrict__ part) {
    constexpr int NT = 64 * NW, W = 64 * CPL, PARTS = 2 * NT / W;
    constexpr int U = W / (NW * R * PARTS);   // products of W rows at once
    static_assert(NT % W == 0, "a thread a column");
    typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
    __shared__ double buf[NW][W];
    __shared__ double z[W + 1], u[W + 1], sh[CPL];
    const int P = b.P, N = b.N, c1 = c + 1, len = N - c1;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int blk0 = c1 / (NW * R);
    if ((int)blockIdx.x < blk0) return;
    // the products first: all loads in flight, two columns each, in the order
    // they are needed (the rows are waited for only after the reflectors)
    const int jp = 2 * (t % (W / 2));
    double s0 = 0.0, s1 = 0.0;
    for (int q = q0 + t / (W / 2); q < ns; q += U * PARTS) {
        pair_t v[U];
#pragma unroll
        for (int e = 0; e < U; ++e) {
            const double* from = src + (long)(q + e * PARTS) * N + c + jp;
            const bool row = q + e * PARTS < ns;
            v[e] = pair_t{0.0, 0.0};
            if (row && jp < len) v[e] = *reinterpret_cast<const pair_t*>(from);
            else if (row && jp == len) v[e].x = *from;
        }
#pragma unroll
        for (int e = 0; e < U; ++e) {
            s0 += v[e].x;
            s1 += v[e].y;
        }
    }
    // column c + tj of row c
    const double* rowc = b.A + (long)c * N;
    const int tj = t % W;
    const double alpha = rowc[c], rj = tj <= len ? rowc[c + tj] : 0.0;
    double* Ai[R];
    bool in[R];
    double a[R][CPL], x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = (blockIdx.x * R + r) * NW + w;
        in[r] = i >= c1 && i < P;
        Ai[r] = b.A + (long)i * N + c1;
        x[r] = in[r] ? Ai[r][-1] : 0.0;
#pragma unroll
        for (int q = 0; q < CPL; ++q) a[r][q] = in[r] && lane + 64 * q < len ? Ai[r][lane + 64 * q] : 0.0;
    }
    buf[t / (W / 2)][jp] = s0;
    buf[t / (W / 2)][jp + 1] = s1;
    __syncthreads();
    double pc = buf[0][0], pj = buf[0][tj];
#pragma unroll
    for (int q = 1; q < PARTS; ++q) {
        pc += buf[q][0];
        pj += buf[q][tj];
    }
    const Refl h = reflector(alpha, pc);
    const double zj = left_part(h, rj, pj), uj = left_rest(rj, zj);
    if (t < W) {
        if (t > 0) {
            z[t - 1] = zj;
            u[t - 1] = uj;
        }
        const double n2 = wave_sum(t > 1 && t <= len ? uj * uj : 0.0);
        if (lane == 0) sh[w] = n2;
    }
    __syncthreads();
    double n2 = sh[0];
#pragma unroll
    for (int q = 1; q < CPL; ++q) n2 += sh[q];
    const Refl k = reflector(len > 0 ? u[0] : 0.0, n2);
    const int ldq = pad16(P), ldp = pad16(N);
    if ((int)blockIdx.x == blk0) {
        double* vq = b.VQ + (long)c * ldq;
        for (int q = t; q <= c; q += NT) vq[q] = q == c ? 1.0 : 0.0;
        for (int q = P + t; q < ldq; q += NT) vq[q] = 0.0;
        if (len > 0) {
            double* vp = b.VP + (long)c * ldp;
            for (int q = t; q < ldp; q += NT)
                vp[q] = q < c1 || q >= N ? 0.0 : q == c1 ? 1.0 : u[q - c1] * k.scale;
        }
        if (t == 0) {
            b.tauq[c] = h.tau;
            b.d[c] = h.beta;
            b.taup[c] = k.tau;
            b.e[c] = k.beta;
        }
    }
    double acc[CPL];
    {
        double zl[CPL], ul[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
            const int j = lane + 64 * q;
            acc[q] = 0.0;
            zl[q] = j < len ? z[j] : 0.0;
            ul[q] = j == 0 ? 1.0 : j < len ? u[j] * k.scale : 0.0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double v = x[r] * h.scale;
            const int i = (blockIdx.x * R + r) * NW + w;
            if (in[r] && lane == 0) b.VQ[(long)c * ldq + i] = v;
            double d = 0.0;
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
                a[r][q] -= v * zl[q];
                d += a[r][q] * ul[q];
            }
            d = k.tau * wave_sum(d);
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
                a[r][q] -= d * ul[q];
                if (in[r] && lane + 64 * q < len) Ai[r][lane + 64 * q] = a[r][q];
            }
            // the next step's column products: rows below its own row
            const double xn = i == c1 || !in[r] ? 0.0 : lane_value(a[r][0], 0);
#pragma unroll
            for (int q = 0; q < CPL; ++q) acc[q] += xn * a[r][q];
        }
    }
#pragma unroll
    for (int q = 0; q < CPL; ++q) buf[w][lane + 64 * q] = acc[q];
    __syncthreads();
    if (t < len) {
        double v = buf[0][t];
#pragma unroll
        for (int q = 1; q < NW; ++q) v += buf[q][t];
        part[(long)blockIdx.x * N + c1 + t] = v;
    }
}

// The sum over the four 16-lane rows of the wavefront for four values at a
// time, scattered: row g ends with the sum of v[{0, 2, 1, 3}[g]] (the swaps
// pair the halves and then the rows of two values, so an addition serves both).
__device__ inline double rows_sum4(double v0, double v1, double v2, double v3) {
    return swap_add16(swap_add32(v0, v1), swap_add32(v2, v3));
}
// The sum over the 16 lanes of each row, returned to all of them.
__device__ inline double row_sum(double v) {
    v += dpp_move<0xB1, 0xf>(v);
    v += dpp_move<0x4E, 0xf>(v);
    v += dpp_move<0x141, 0xf>(v);
    v += dpp_move<0x140, 0xf>(v);
    return v;
}

// The rest of the bidiagonalisation from column c0 on by one workgroup, the
// trailing block (at most 4 NW RS rows, 16 CS columns) in its registers: lane
// (g, cx) of wavefront w holds the rows 4 w + g + 4 NW s and the columns
// cx + 16 u.  A step costs two barriers: the products of column c with every
// column (with itself: its norm) are summed over the wavefronts in LDS, and
// row c goes with them, so that after them every lane has its part of the
// updated row c, from which the right reflector follows without another
// exchange (the sums along a row stay inside 16 lanes).
template <int NW, int RS, int CS>
struct TailLDS {
    double part[NW][16 * CS], psum[16 * CS], rowc[2][16 * CS], colc[2][4 * NW * RS];
};

// Columns 16 U0 .. 16 U0 + 15 of it.
template <int NW, int RS, int CS, int U0>
__device__ __forceinline__ void bd_tail_columns(const BdWork& b, int c0, double (&a)[RS][CS],
                                                TailLDS<NW, RS, CS>& L) {
    constexpr int RW = 4 * NW, NC = 16 * CS;         // rows and columns a register slot covers in all
    constexpr int s0 = U0 * 16 / RW;                 // row slots before it are finished
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, cx = lane & 15, g = lane >> 4, ry = 4 * w + g;
    const int P = b.P, N = b.N, C = N - c0;
    const int sel = ((g & 1) << 1) | (g >> 1);       // the slot of four whose sum this row of lanes gets
    const int cols = min(16, C - 16 * U0);
    for (int cc = 0; cc < cols; ++cc) {
        const int c = 16 * U0 + cc;
        double* rowc = L.rowc[c & 1];
        double* colc = L.colc[c & 1];
        // column c below row c, to every lane of a row (and to LDS)
        double x[RS];
#pragma unroll
        for (int s = s0; s < RS; ++s) {
            const double v = __shfl(a[s][U0], cc, 16);
            x[s] = ry + RW * s > c ? v : 0.0;
        }
        if (cx == cc) {
#pragma unroll
            for (int s = s0; s < RS; ++s) colc[ry + RW * s] = x[s];
        }
        if (ry == c % RW) {
#pragma unroll
            for (int u = U0; u < CS; ++u) rowc[cx + 16 * u] = a[s0][u];
        }
        // the products of column c with the columns from c on
#pragma unroll
        for (int u = U0 & ~3; u < CS; u += 4) {
            double v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q] = 0.0;
                if (u + q >= U0) {
#pragma unroll
                    for (int s = s0; s < RS; ++s) v[q] += x[s] * a[s][u + q];
                }
            }
            L.part[w][16 * (u + sel) + cx] = rows_sum4(v[0], v[1], v[2], v[3]);
        }
        __syncthreads();
        if (t < NC) {
            double p = L.part[0][t];
#pragma unroll
            for (int q = 1; q < NW; ++q) p += L.part[q][t];
            L.psum[t] = p;
        }
        double sg = L.part[0][c];
#pragma unroll
        for (int q = 1; q < NW; ++q) sg += L.part[q][c];
        const Refl h = reflector(rowc[c], sg);
        __syncthreads();
        double r[CS];
#pragma unroll
        for (int s = s0; s < RS; ++s) x[s] *= h.scale;
#pragma unroll
        for (int u = U0; u < CS; ++u) {
            const int j = cx + 16 * u;
            const double rc = rowc[j], z = left_part(h, rc, L.psum[j]);
            r[u] = left_rest(rc, z);
#pragma unroll
            for (int s = s0; s < RS; ++s) a[s][u] -= x[s] * z;
        }
        // the reflector's row of VQ, a value a thread
        const int ldq = pad16(P), ldp = pad16(N);
        for (int i = t; i < ldq; i += 64 * NW) {
            const int l = i - c0;
            b.VQ[(long)(c0 + c) * ldq + i] = l < c || i >= P ? 0.0 : (l == c ? 1.0 : h.scale * colc[l]);
        }
        if (t == 0) {
            b.tauq[c0 + c] = h.tau;
            b.d[c0 + c] = h.beta;
        }
        if (c + 1 >= C) return;
        // right reflector from the updated row c
        double n2 = 0.0;
#pragma unroll
        for (int u = U0; u < CS; ++u) n2 += cx + 16 * u > c + 1 ? r[u] * r[u] : 0.0;
        n2 = row_sum(n2);
        const double alpha = __shfl(cc < 15 ? r[U0] : r[U0 + 1 < CS ? U0 + 1 : U0], (c + 1) & 15, 16);
        const Refl k = reflector(alpha, n2);
#pragma unroll
        for (int u = U0; u < CS; ++u) {
            const int j = cx + 16 * u;
            r[u] = j > c + 1 ? r[u] * k.scale : (j == c + 1 ? 1.0 : 0.0);
        }
        // (rows up to c are finished: their registers are not read again)
#pragma unroll
        for (int s = s0; s < RS; ++s) {
            double q = 0.0;
#pragma unroll
            for (int u = U0; u < CS; ++u) q += a[s][u] * r[u];
            q = k.tau * row_sum(q);
#pragma unroll
            for (int u = U0; u < CS; ++u) a[s][u] -= q * r[u];
        }
        // the row of VP, from the registers of one row of lanes (formed anew it
        // would have to round alike: next to nothing is left of a row that is
        // almost finished)
        double* vp = b.VP + (long)(c0 + c) * ldp;
        if (ry == c % RW) {
#pragma unroll
            for (int u = U0; u < CS; ++u)
                if (c0 + cx + 16 * u < ldp) vp[c0 + cx + 16 * u] = r[u];
        }
        for (int j = t; j < c0 + 16 * U0; j += 64 * NW) vp[j] = 0.0;
        for (int j = c0 + NC + t; j < ldp; j += 64 * NW) vp[j] = 0.0;
        if (t == 0) {
            b.taup[c0 + c] = k.tau;
            b.e[c0 + c] = k.beta;
        }
    }
}

template <int NW, int RS, int CS, int U0>
__device__ __forceinline__ void bd_tail_from(const BdWork& b, int c0, double (&a)[RS][CS],
                                             TailLDS<NW, RS, CS>& L) {
    if constexpr (U0 < CS) {
        bd_tail_columns<NW, RS, CS, U0>(b, c0, a, L);
        bd_tail_from<NW, RS, CS, U0 + 1>(b, c0, a, L);
    }
}

// c0 = 0: the block may be theta itself (tr: its transpose), and the padding
// rows of the reflectors are cleared here.
template <int NW, int RS, int CS>
__global__ __launch_bounds__(64 * NW) void bd_tail_kernel(BdWork b, int c0, const double* __restrict__ theta, int tr) {
    constexpr int RW = 4 * NW;
    static_assert(RW % 16 == 0 && CS % 4 == 0 && 16 * CS <= 64 * NW, "slots");
    __shared__ TailLDS<NW, RS, CS> L;
    const int t = threadIdx.x, lane = t & 63, cx = lane & 15, ry = 4 * (t >> 6) + (lane >> 4);
    const int R = b.P - c0, C = b.N - c0;
    double a[RS][CS];
#pragma unroll
    for (int s = 0; s < RS; ++s)
#pragma unroll
        for (int u = 0; u < CS; ++u) {
            const int i = ry + RW * s, j = cx + 16 * u;
            const bool in = i < R && j < C;
            if (theta) a[s][u] = in ? theta[tr ? (long)j * b.P + i : (long)i * b.N + j] : 0.0;
            else a[s][u] = in ? b.A[(long)(c0 + i) * b.N + c0 + j] : 0.0;
        }
    if (theta) clear_padding(b.P, b.N, b.VQ, b.VP, t, 64 * NW);
    bd_tail_from<NW, RS, CS, 0>(b, c0, a, L);
}

// The triangular factors of the reflector blocks: H_0 ... H_15 = I - V T V^T,
// T_jj = tau_j, T[0:j, j] = -tau_j T[0:j, 0:j] (V^T v_j); stored as -T.  Grid: block x side (0: VQ, 1: VP).
__global__ __launch_bounds__(256) void wy_t_kernel(const double* __restrict__ VQ, int P, const double* __restrict__ VP,
                                                   int N, const double* __restrict__ tauq,
                                                   const double* __restrict__ taup, double* __restrict__ TQ,
                                                   double* __restrict__ TP) {
    __shared__ double Sp[4][WYB][WYB + 1];
    __shared__ double S[WYB][WYB + 1];
    const int side = blockIdx.y, b0 = blockIdx.x * WYB;
    const int len = pad16(side ? N : P), nr = side ? N - 1 : N;
    const double* V = side ? VP : VQ;
    const double* tau = side ? taup : tauq;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, l16 = lane & 15, kg = lane >> 4;
    const double* v = V + (long)(b0 + l16) * len;
    d4_t acc = {0, 0, 0, 0};
    for (int k0 = b0 + 4 * w; k0 < len; k0 += 16) {
        const double x = v[k0 + kg];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x, x, acc, 0, 0, 0);
    }
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) Sp[w][4 * rr + kg][l16] = acc[rr];
    __syncthreads();
    {
        const int i = t >> 4, j = t & 15;
        S[i][j] = (Sp[0][i][j] + Sp[1][i][j]) + (Sp[2][i][j] + Sp[3][i][j]);
    }
    __syncthreads();
    if (t < WYB) {
        double trow[WYB];
        double* T = (side ? TP : TQ) + (long)blockIdx.x * WYB * WYB + t * WYB;
#pragma unroll
        for (int j = 0; j < WYB; ++j) {
            const double tj = b0 + j < nr ? tau[b0 + j] : 0.0;
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < j; ++k) s += trow[k] * S[k][j];
            trow[j] = t < j ? -tj * s : (t == j ? tj : 0.0);
            T[j] = -trow[j];
        }
    }
}

// Vector t < k of a side: H_0 H_1 ... (the reflectors V, nblk blocks of 16
// with rows of pad16(len)) applied to row perm[t] of X [n][n] (zero-extended
// to len), times sg[perm[t]] *scale
// when scaled; written to out[t][len], or transposed to out[len][k].
struct WySide {
    const double* X;
    const double* V;
    const double* T;       // -T of the blocks
    int len, nblk;
    double* out;
    double* tmp;      // [pad16(k)][pad16(len)], only for len > the register limit
    int transposed, scaled;
};

// NW wavefronts hold 16 vectors; wavefront w owns the 16-column tiles w,
// w + NW, ... of them, TPW in registers (TPW = 0: any number, kept in tmp).
// Per reflector block from the last to the first: W = V^T x (partials of the
// wavefronts summed in LDS in a fixed order), W2 = T W, x -= V W2.  Tiles
// before the block's first reflector are untouched.
template <int NW, int TPW>
__global__ __launch_bounds__(64 * NW) void wy_apply_kernel(WySide s0, WySide s1, int n, const int* __restrict__ perm,
                                                           int k, const double* __restrict__ sg,
                                                           const double* __restrict__ scale) {
    __shared__ double Wp[NW][4][64];
    __shared__ double Ws[WYB][WYB + 1];
    constexpr int TR = TPW > 0 ? TPW : 1;
    const WySide s = blockIdx.y ? s1 : s0;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int vec = blockIdx.x * WYB + l16;       // this lane's vector
    const int row = vec < k ? perm[vec] : -1;
    const int ld = pad16(s.len), ntile = ld / WYB, nblk = s.nblk;
    double* tmp = TPW > 0 ? nullptr : s.tmp + (long)vec * ld;
    d4_t acc[TR];
    auto first = [&](int tile, d4_t& x) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int c = tile * WYB + 4 * rr + kg;
            x[rr] = (row >= 0 && c < n) ? s.X[(long)row * n + c] : 0.0;
        }
    };
    auto load = [&](int tile, d4_t& x) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) x[rr] = tmp[tile * WYB + 4 * rr + kg];
    };
    auto store = [&](int tile, const d4_t& x) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) tmp[tile * WYB + 4 * rr + kg] = x[rr];
    };
    // Operands of a block: its reflectors as rows (W) and as columns (the
    // update), and T.
    auto load_dot = [&](int b, int tile, double (&a)[4]) {
        const double* v = s.V + (long)(b * WYB + l16) * ld + tile * WYB + kg;
#pragma unroll
        for (int st = 0; st < 4; ++st) a[st] = v[4 * st];
    };
    auto load_upd = [&](int b, int tile, double (&a)[4]) {
        const double* v = s.V + (long)(b * WYB + kg) * ld + tile * WYB + l16;
#pragma unroll
        for (int st = 0; st < 4; ++st) a[st] = v[(long)(4 * st) * ld];
    };
    auto load_t = [&](int b, double (&a)[4]) {
#pragma unroll
        for (int st = 0; st < 4; ++st) a[st] = s.T[(long)b * WYB * WYB + l16 * WYB + 4 * st + kg];
    };
    auto mma4 = [](const double (&a)[4], const d4_t& x, d4_t c) {
#pragma unroll
        for (int st = 0; st < 4; ++st) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[st], x[st], c, 0, 0, 0);
        return c;
    };
    // Up to 512 entries the operands are fetched as soon as the block before has
    // used its own, across the barriers, and every tile takes
    // part in every block (it meets zeros before a block's first reflector).
    constexpr bool PF = TPW > 0 && NW * TPW <= 32;
    int tl[TR];
#pragma unroll
    for (int u = 0; u < TR; ++u) tl[u] = PF ? min(w + NW * u, ntile - 1) : w + NW * u;
    double vd[PF ? TR : 1][4], vu[PF ? TR : 1][4], tt[4];
    if (TPW > 0) {
#pragma unroll
        for (int u = 0; u < TR; ++u) {
            acc[u] = d4_t{0, 0, 0, 0};
            if (w + NW * u < ntile) first(w + NW * u, acc[u]);
        }
    } else {
        for (int tile = w; tile < ntile; tile += NW) {
            d4_t x;
            first(tile, x);
            store(tile, x);
        }
    }
    if (PF) {
        // the reflectors into this XCD's L2 first, one load a cache line with
        // many in flight, so that a block waits for L2 and not for memory
        double warm = 0.0;
        const int lines = nblk * ld;      // 16 ld values a block, 16 a line
        for (int e = t; e < lines; e += 64 * NW) warm += s.V[(long)e * 16];
        asm volatile("" ::"v"(warm));
#pragma unroll
        for (int u = 0; u < (PF ? TR : 0); ++u) {
            load_dot(nblk - 1, tl[u], vd[u]);
            load_upd(nblk - 1, tl[u], vu[u]);
        }
        load_t(nblk - 1, tt);
    }
    for (int b = nblk - 1; b >= 0; --b) {
        const int bn = max(b - 1, 0);
        // W = V^T x over this wavefront's tiles
        d4_t wp = {0, 0, 0, 0};
        if (PF) {
#pragma unroll
            for (int u = 0; u < (PF ? TR : 0); ++u) {
                wp = mma4(vd[u], acc[u], wp);
                load_dot(bn, tl[u], vd[u]);
            }
        } else if (TPW > 0) {
#pragma unroll
            for (int u = 0; u < TR; ++u) {
                if (tl[u] < b || tl[u] >= ntile) continue;
                double a[4];
                load_dot(b, tl[u], a);
                wp = mma4(a, acc[u], wp);
            }
        } else {
            for (int tile = w; tile < ntile; tile += NW) {
                if (tile < b) continue;
                d4_t x;
                double a[4];
                load(tile, x);
                load_dot(b, tile, a);
                wp = mma4(a, x, wp);
            }
        }
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) Wp[w][rr][lane] = wp[rr];
        __syncthreads();
        for (int e = t; e < WYB * WYB; e += 64 * NW) {
            // accumulator element rr of lane (kg, l16): reflector 4 rr + kg, vector l16
            const int i = e >> 4, v = e & 15, rr = i >> 2, ln = (i & 3) * 16 + v;
            double sum = Wp[0][rr][ln];
#pragma unroll
            for (int q = 1; q < NW; ++q) sum += Wp[q][rr][ln];
            Ws[i][v] = sum;
        }
        __syncthreads();
        if (!PF) load_t(b, tt);
        d4_t ws, w2 = {0, 0, 0, 0};
#pragma unroll
        for (int st = 0; st < 4; ++st) ws[st] = Ws[4 * st + kg][l16];
        w2 = mma4(tt, ws, w2);
        if (PF) {
            load_t(bn, tt);
#pragma unroll
            for (int u = 0; u < (PF ? TR : 0); ++u) {
                if (w + NW * u < ntile) acc[u] = mma4(vu[u], w2, acc[u]);
                load_upd(bn, tl[u], vu[u]);
            }
        } else if (TPW > 0) {
#pragma unroll
            for (int u = 0; u < TR; ++u) {
                if (tl[u] < b || tl[u] >= ntile) continue;
                double a[4];
                load_upd(b, tl[u], a);
                acc[u] = mma4(a, w2, acc[u]);
            }
        } else {
            for (int tile = w; tile < ntile; tile += NW) {
                if (tile < b) continue;
                d4_t x;
                double a[4];
                load(tile, x);
                load_upd(b, tile, a);
                store(tile, mma4(a, w2, x));
            }
        }
    }
    if (row < 0) return;
    const double f = s.scaled ? sg[row] * *scale : 1.0;
    auto put = [&](int tile, const d4_t& x) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int cc = tile * WYB + 4 * rr + kg;
            if (cc >= s.len) continue;
            if (s.transposed) s.out[(long)cc * k + vec] = f * x[rr];
            else s.out[(long)vec * s.len + cc] = f * x[rr];
        }
    };
    if (TPW > 0) {
#pragma unroll
        for (int u = 0; u < TR; ++u)
            if (w + NW * u < ntile) put(w + NW * u, acc[u]);
    } else {
        for (int tile = w; tile < ntile; tile += NW) {
            d4_t x;
            load(tile, x);
            put(tile, x);
        }
    }
}

// Rows of the block that one workgroup finishes: a column takes it 2 us where a step
// takes 5, so as many as it holds in registers (72 doubles a lane, 144 of its 256
// registers; 256 rows would need them all).  Its three shapes by what is left, us for
// a whole block in this shape and in the next larger: 32 rows 44 and 68, 64 76 and 117
// (4, 4, 4); 80 138 and 218, 128 191 and 304 (4, 8, 8).
constexpr int BD_TAIL = 192;
constexpr int BD_ONE = 512;                 // rows and columns from which on a step is one launch
constexpr int WY_MAX = 8 * WYB * 16;     // longest vector held in registers

}  // namespace

size_t bd_workspace(int P, int N) {
    const size_t nb = (size_t)(N + WYB - 1) / WYB, np = pad16(N);
    return (size_t)P * N + np * pad16(P) + np * np + 2 * nb * WYB * WYB +
           2 * (size_t)((P + 15) / 16) * N + 5 * (size_t)N + 64;
}

BdWork bd_carve(double* ws, int P, int N) {
    BdWork w{};
    const size_t nb = (size_t)(N + WYB - 1) / WYB;
    w.P = P;
    w.N = N;
    w.A = ws;
    w.VQ = w.A + (size_t)P * N;
    w.VP = w.VQ + (size_t)pad16(N) * pad16(P);
    w.TQ = w.VP + (size_t)pad16(N) * pad16(N);
    w.TP = w.TQ + nb * WYB * WYB;
    w.part = w.TP + nb * WYB * WYB;
    w.p = w.part + 2 * (size_t)((P + 15) / 16) * N;
    w.tauq = w.p + N;
    w.taup = w.tauq + N;
    w.d = w.taup + N;
    w.e = w.d + N;
    return w;
}

void bidiagonalise(const BdWork& w, const double* theta, bool tr, hipStream_t s, LaunchProbe* probe) {
    const int P = w.P, N = w.N;
    auto step = [&](int c, bool start) {
        const bool timed = probe && probe->begin(PK_BIDIAG, s);
        const int len = N - c - 1, g = (P + BS_NW - 1) / BS_NW;
        const dim3 grid(g), block(BS_NT);
        if (len <= 512) hipLaunchKernelGGL((bd_step_kernel<1>), grid, block, 0, s, w, c, start);
        else if (len <= 1024) hipLaunchKernelGGL((bd_step_kernel<2>), grid, block, 0, s, w, c, start);
        else if (len <= 2048) hipLaunchKernelGGL((bd_step_kernel<4>), grid, block, 0, s, w, c, start);
        else hipLaunchKernelGGL(bd_step_long_kernel, grid, block, 0, s, w, c, start);
        if (len > 0) hipLaunchKernelGGL(bd_sum_kernel, dim3((len + 15) / 16), dim3(1024), 0, s, w, c + 1,
                                        (c + 1) / BS_NW, g);
        if (timed) probe->end(PK_BIDIAG, s);
    };
    // the products of the column the next step clears: in p (ns = 1), or a row
    // per workgroup in one half of part while the steps take one launch each
    const double* src = w.p;
    int q0 = 0, ns = 1;
    double* const half[2] = {w.part, w.part + (size_t)((P + 15) / 16) * N};
    auto step1 = [&](int c) {
        const bool timed = probe && probe->begin(PK_BIDIAG, s);
        double* out = half[c & 1];
        constexpr int NW = 8, R = 2;
        const int g = (P + NW * R - 1) / (NW * R);
#define ITE_S1(CPL) \
    hipLaunchKernelGGL((bd_step1_kernel<CPL, R, NW>), dim3(g), dim3(64 * NW), 0, s, w, c, src, q0, ns, out)
        if (N - c <= 256) ITE_S1(4);
        else ITE_S1(8);
#undef ITE_S1
        src = out;
        q0 = (c + 1) / (NW * R);
        ns = g;
        if (timed) probe->end(PK_BIDIAG, s);
    };
    const bool whole = P <= BD_TAIL;
    if (!whole) {
        hipLaunchKernelGGL(bd_load_kernel, dim3((N + 31) / 32, (P + 31) / 32), dim3(256), 0, s, theta, P, N, (int)tr,
                           w.A, w.VQ, w.VP);
        step(-1, true);
    }
    for (int c = 0; c < N; ++c) {
        const int len = P - c;
        if (len > BD_TAIL) {
            if (N - c <= BD_ONE && len <= BD_ONE) step1(c);
            else step(c, false);
            continue;
        }
        const bool timed = probe && probe->begin(PK_BIDIAG, s);
        const double* th = whole ? theta : nullptr;
#define ITE_TAIL(NW, RS, CS) \
    hipLaunchKernelGGL((bd_tail_kernel<NW, RS, CS>), dim3(1), dim3(64 * NW), 0, s, w, c, th, (int)tr)
        if (len <= 64) ITE_TAIL(4, 4, 4);
        else if (len <= 128) ITE_TAIL(4, 8, 8);
        else ITE_TAIL(8, 6, 12);
#undef ITE_TAIL
        if (timed) probe->end(PK_BIDIAG, s);
        break;
    }
    hipLaunchKernelGGL(wy_t_kernel, dim3((N + WYB - 1) / WYB, 2), dim3(256), 0, s, w.VQ, P, w.VP, N, w.tauq, w.taup,
                       w.TQ, w.TP);
    HIP_CHECK(hipGetLastError());
    if (probe) {
        // 4 P N^2 - 4 N^3 / 3 flops; the block read and the reflectors written,
        // and the trailing block read and written by every step before the tail
        const double p = P, n = N;
        double bytes = 8.0 * (2.0 * p * n + n * n);
        for (int c = 0; c < N && P - c > BD_TAIL; ++c) bytes += 16.0 * (P - c) * (N - c - 1);
        probe->work(PK_BIDIAG, 4.0 * n * n * (p - n / 3.0), bytes);
    }
}

void bd_vectors(const BdWork& w, const double* XQ, const double* XP, const int* perm, int k, const double* sg,
                const double* scale, const BdOut& q, const BdOut& p, double* tmp, hipStream_t s, LaunchProbe* probe) {
    if (k <= 0) return;
    const int N = w.N;
    const int kr = pad16(k);
    const int nblk = (N + WYB - 1) / WYB;
    WySide sq{XQ, w.VQ, w.TQ, w.P, nblk, q.out, tmp, q.transposed, q.scaled};
    WySide sp{XP, w.VP, w.TP, N, nblk, p.out, tmp ? tmp + (size_t)kr * pad16(w.P) : nullptr, p.transposed, p.scaled};
    const dim3 grid(kr / WYB, 2);
    const bool timed = probe && probe->begin(PK_VECTORS, s);
    const int tiles = (w.P + WYB - 1) / WYB;
// By tiles of 16 entries: as few wavefronts as hold them, since each has a part of
// every block's sum and its own copy of T W.  us for half the vectors (32 and 64 rows:
// all) of n x n blocks, the shape taken and the next ones:
//      n      4,1   4,2   4,4   8,4   8,8  16,4  8,16   8,0
//      64    10.5  12.8  18.1  30.9
//      128         20.6  30.5  53.2
//      256               57.2  99.9
//      320                      124    74    87    82
//      512                      199   144   167   157
//      600                            185   207   202   392
//      1024                           427   461   452   956
//      2048                                      1495  3661
// (8 wavefronts of 8 tiles, the fastest from 320 to 1024 rows, are not built yet.)
#define ITE_WY(NW, TPW) \
    hipLaunchKernelGGL((wy_apply_kernel<NW, TPW>), grid, dim3(64 * NW), 0, s, sq, sp, N, perm, k, sg, scale)
    if (tiles <= 4) ITE_WY(4, 1);
    else if (tiles <= 8) ITE_WY(4, 2);
    else if (tiles <= 16) ITE_WY(4, 4);
    else if (tiles <= 32) ITE_WY(8, 4);
    else if (tiles <= 64) ITE_WY(16, 4);
    else if (tiles <= WY_MAX / WYB) ITE_WY(8, 16);
    else ITE_WY(8, 0);
#undef ITE_WY
    if (timed) probe->end(PK_VECTORS, s);
    HIP_CHECK(hipGetLastError());
    if (probe) {
        // per vector and reflector: a dot product and an update over its entries
        const double pq = w.P, n = N;
        probe->work(PK_VECTORS, 4.0 * k * n * ((pq - n / 2.0) + n / 2.0), 8.0 * ((pq + n) * (n / 2.0 + 2.0 * k)));
    }
}

size_t bd_vectors_tmp(int P, int N, int k) {
    if (P <= WY_MAX) return 0;
    return (size_t)pad16(k) * ((size_t)pad16(P) + pad16(N));
}

}  // namespace ite
