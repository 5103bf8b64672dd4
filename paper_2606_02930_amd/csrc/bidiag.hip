// Householder bidiagonalisation of a two-site block and the way back from
// the singular vectors of the bidiagonal matrix to those of the block.
//
// A (P x N, P >= N, row-major) becomes B = Q^T A Z, upper bidiagonal (Golub
// and Kahan): in step c a reflector on the rows from c on clears column c
// below the diagonal, one on the columns from c + 1 on clears row c right of
// the superdiagonal.  One launch applies the left reflector (workgroups own
// 16-column strips: the products v^T A of a strip need no other workgroup),
// the next the right one (a wavefront owns a row).  Each launch leaves the row
// or column that the next reflector is formed from in a contiguous buffer,
// and every workgroup forms that reflector for itself, in the same order, so
// that two launches a step are all the synchronisation there is.
//
// The reflectors are kept as rows (VQ [N][P], VP [N][N]; zero before the
// first entry, which is one).  bd_vectors applies them in blocks of 16 in the
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

// The reflector of x[0..len) (LAPACK's convention: beta = -sign(alpha) ||x||,
// tau = (beta - alpha) / beta, v = x / (alpha - beta) with v_0 = 1; tau = 0
// when x_1.. = 0).  Every thread of the workgroup gets it; sh: one double per
// wavefront.
struct Refl {
    double beta, tau, scale;
};
__device__ inline Refl reflector(double alpha, double sg) {
    Refl r{alpha, 0.0, 0.0};
    if (sg > 0.0) {
        const double nrm = sqrt(alpha * alpha + sg);
        r.beta = alpha >= 0.0 ? -nrm : nrm;
        r.tau = (r.beta - alpha) / r.beta;
        r.scale = 1.0 / (alpha - r.beta);
    } else if (!(sg == 0.0)) {
        r.beta = r.tau = sg;     // NaN stays visible in the result
    }
    return r;
}
template <int NT>
__device__ inline Refl block_reflector(const double* __restrict__ x, int len, double* sh) {
    double sg = 0.0;
    for (int i = 1 + threadIdx.x; i < len; i += NT) sg += x[i] * x[i];
    sg = wave_sum(sg);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = sg;
    __syncthreads();
    sg = sh[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) sg += sh[w];
    return reflector(x[0], sg);
}

// A <- theta (P x N), or theta^T when tr (theta then N x P); col <- column 0.
__global__ __launch_bounds__(256) void bd_load_kernel(const double* __restrict__ theta, int P, int N, int tr,
                                                      double* __restrict__ A, double* __restrict__ col) {
    __shared__ double tile[32][33];
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
        const double v = tr ? tile[y][x] : theta[(long)r * N + c];
        A[(long)r * N + c] = v;
        if (c == 0) col[r] = v;
    }
}

// Left reflector of step c from col[c..P), applied to the columns c + 1..;
// row[j] <- A[c][j].  16 columns a workgroup; thread (tx, ty) keeps the rows
// c + ty, c + ty + NT / 16, ... of its column in registers when there are at
// most RPT of them, so A is read and written once.
template <int NT, int RPT>
__global__ __launch_bounds__(NT) void bd_left_kernel(double* __restrict__ A, int P, int N, int c,
                                                     const double* __restrict__ col, double* __restrict__ row,
                                                     double* __restrict__ VQ, double* __restrict__ tauq,
                                                     double* __restrict__ d) {
    constexpr int RG = NT / 16, NW = NT / 64;
    __shared__ double sh[NW];
    __shared__ double part[NW][16];
    const int t = threadIdx.x, tx = t & 15, ty = t >> 4;
    const int len = P - c;
    const int j = c + 1 + blockIdx.x * 16 + tx;
    const bool in = j < N;
    const bool keep = len <= RG * RPT;
    double a[RPT];
    double* Aj = A + (long)c * N + j;
    if (keep) {
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int i = ty + RG * u;
            a[u] = (in && i < len) ? Aj[(long)i * N] : 0.0;
        }
    }
    const double* x = col + c;
    const Refl h = block_reflector<NT>(x, len, sh);
    if (blockIdx.x == 0) {
        double* v = VQ + (long)c * P;
        for (int i = t; i < P; i += NT) v[i] = i < c ? 0.0 : (i == c ? 1.0 : col[i] * h.scale);
        if (t == 0) {
            tauq[c] = h.tau;
            d[c] = h.beta;
        }
    }
    double z = 0.0;
    if (keep) {
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int i = ty + RG * u;
            if (i < len) z += (i == 0 ? 1.0 : x[i] * h.scale) * a[u];
        }
    } else if (in) {
        for (int i = ty; i < len; i += RG) z += (i == 0 ? 1.0 : x[i] * h.scale) * Aj[(long)i * N];
    }
    z += __shfl_xor(z, 16, 64);
    z += __shfl_xor(z, 32, 64);
    if ((t & 63) < 16) part[t >> 6][tx] = z;
    __syncthreads();
    z = part[0][tx];
#pragma unroll
    for (int w = 1; w < NW; ++w) z += part[w][tx];
    z *= h.tau;
    if (!in) return;
    if (keep) {
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int i = ty + RG * u;
            if (i >= len) continue;
            const double v = a[u] - (i == 0 ? 1.0 : x[i] * h.scale) * z;
            if (i == 0) row[j] = v;
            else Aj[(long)i * N] = v;
        }
    } else {
        for (int i = ty; i < len; i += RG) {
            const double v = Aj[(long)i * N] - (i == 0 ? 1.0 : x[i] * h.scale) * z;
            if (i == 0) row[j] = v;
            else Aj[(long)i * N] = v;
        }
    }
}

// Right reflector of step c from row[c + 1..N), applied to the rows c + 1..P;
// col[i] <- A[i][c + 1].  A wavefront owns a row and keeps it in registers
// when it has at most 64 CPL columns left.
template <int CPL>
__global__ __launch_bounds__(256) void bd_right_kernel(double* __restrict__ A, int P, int N, int c,
                                                       double* __restrict__ col, const double* __restrict__ row,
                                                       double* __restrict__ VP, double* __restrict__ taup,
                                                       double* __restrict__ e) {
    __shared__ double sh[4];
    const int t = threadIdx.x, lane = t & 63;
    const int c1 = c + 1, len = N - c1;
    const int i = c1 + blockIdx.x * 4 + (t >> 6);
    const bool in = i < P;
    const bool keep = len <= 64 * CPL;
    double* Ai = A + (long)i * N + c1;
    double a[CPL];
    if (keep) {
#pragma unroll
        for (int u = 0; u < CPL; ++u) a[u] = (in && lane + 64 * u < len) ? Ai[lane + 64 * u] : 0.0;
    }
    const double* x = row + c1;
    const Refl h = block_reflector<256>(x, len, sh);
    if (blockIdx.x == 0) {
        double* v = VP + (long)c * N;
        for (int k = t; k < N; k += 256) v[k] = k < c1 ? 0.0 : (k == c1 ? 1.0 : row[k] * h.scale);
        if (t == 0) {
            taup[c] = h.tau;
            e[c] = h.beta;
        }
    }
    if (!in) return;
    double w = 0.0;
    if (keep) {
        double v[CPL];
#pragma unroll
        for (int u = 0; u < CPL; ++u) {
            const int k = lane + 64 * u;
            v[u] = k < len ? (k == 0 ? 1.0 : x[k] * h.scale) : 0.0;
            w += v[u] * a[u];
        }
        w = h.tau * wave_sum(w);
#pragma unroll
        for (int u = 0; u < CPL; ++u) {
            const int k = lane + 64 * u;
            const double r = a[u] - w * v[u];
            if (k < len) Ai[k] = r;
            if (k == 0) col[i] = r;
        }
    } else {
        for (int k = lane; k < len; k += 64) w += (k == 0 ? 1.0 : x[k] * h.scale) * Ai[k];
        w = h.tau * wave_sum(w);
        for (int k = lane; k < len; k += 64) {
            const double r = Ai[k] - w * (k == 0 ? 1.0 : x[k] * h.scale);
            Ai[k] = r;
            if (k == 0) col[i] = r;
        }
    }
}

// The triangular factors T [WYB][WYB] of the reflector blocks:
// H_0 ... H_15 = I - V T V^T, T_jj = tau_j,
// T[0:j, j] = -tau_j T[0:j, 0:j] (V^T v_j).  Grid: block x side (0: VQ, 1: VP).
__global__ __launch_bounds__(256) void wy_t_kernel(const double* __restrict__ VQ, int P, const double* __restrict__ VP,
                                                   int N, const double* __restrict__ tauq,
                                                   const double* __restrict__ taup, double* __restrict__ TQ,
                                                   double* __restrict__ TP) {
    __shared__ double Sp[4][WYB][WYB + 1];
    __shared__ double S[WYB][WYB + 1];
    const int side = blockIdx.y, b0 = blockIdx.x * WYB;
    const int len = side ? N : P, nr = side ? N - 1 : N;
    const double* V = side ? VP : VQ;
    const double* tau = side ? taup : tauq;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, l16 = lane & 15, kg = lane >> 4;
    const bool live = b0 + l16 < nr;
    const double* v = V + (long)(b0 + l16) * len;
    d4_t acc = {0, 0, 0, 0};
    for (int k0 = (b0 & ~3) + 4 * w; k0 < len; k0 += 16) {
        const double x = (live && k0 + kg < len) ? v[k0 + kg] : 0.0;
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
            T[j] = trow[j];
        }
    }
}

// Vector t < k of a side: H_0 H_1 ... (the reflectors V [nr][len]) applied
// to row perm[t] of X [n][n] (zero-extended to len), times sg[perm[t]] *scale
// when scaled; written to out[t][len], or transposed to out[len][k].
struct WySide {
    const double* X;
    const double* V;
    const double* T;
    int len, nr;
    double* out;
    double* tmp;      // [16 ceil(k / 16)][len], only for len > the register limit
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
    const int ntile = (s.len + WYB - 1) / WYB;
    double* tmp = TPW > 0 ? nullptr : s.tmp + (long)vec * s.len;
    d4_t acc[TR];
    if (TPW > 0) {
#pragma unroll
        for (int u = 0; u < TR; ++u)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int c = (w + NW * u) * WYB + 4 * rr + kg;
                acc[u][rr] = (row >= 0 && c < n) ? s.X[(long)row * n + c] : 0.0;
            }
    } else {
        for (int c = w * WYB; c < s.len; c += NW * WYB)
            for (int rr = 0; rr < 4; ++rr) {
                const int cc = c + 4 * rr + kg;
                if (cc < s.len) tmp[cc] = (row >= 0 && cc < n) ? s.X[(long)row * n + cc] : 0.0;
            }
    }
    auto load = [&](int tile, d4_t& x) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int cc = tile * WYB + 4 * rr + kg;
            x[rr] = cc < s.len ? tmp[cc] : 0.0;
        }
    };
    for (int b = (s.nr + WYB - 1) / WYB - 1; b >= 0; --b) {
        const int b0 = b * WYB;
        const double* V = s.V + (long)b0 * s.len;
        const bool live = b0 + l16 < s.nr;
        // W = V^T x over this wavefront's tiles
        d4_t wp = {0, 0, 0, 0};
        auto dot_tile = [&](int tile, const d4_t& x) {
            double a[4];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                const int cc = tile * WYB + 4 * st + kg;
                a[st] = (live && cc < s.len) ? V[(long)l16 * s.len + cc] : 0.0;
            }
#pragma unroll
            for (int st = 0; st < 4; ++st) wp = __builtin_amdgcn_mfma_f64_16x16x4f64(a[st], x[st], wp, 0, 0, 0);
        };
        if (TPW > 0) {
#pragma unroll
            for (int u = 0; u < TR; ++u) {
                const int tile = w + NW * u;
                if (tile >= b && tile < ntile) dot_tile(tile, acc[u]);
            }
        } else {
            for (int tile = w; tile < ntile; tile += NW) {
                if (tile < b) continue;
                d4_t x;
                load(tile, x);
                dot_tile(tile, x);
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
        d4_t w2 = {0, 0, 0, 0};
        const double* T = s.T + (long)b * WYB * WYB;
#pragma unroll
        for (int st = 0; st < 4; ++st)
            w2 = __builtin_amdgcn_mfma_f64_16x16x4f64(-T[l16 * WYB + 4 * st + kg], Ws[4 * st + kg][l16], w2, 0, 0, 0);
        auto update_tile = [&](int tile, d4_t& x) {
            const int cc = tile * WYB + l16;
            double a[4];
#pragma unroll
            for (int st = 0; st < 4; ++st)
                a[st] = (b0 + 4 * st + kg < s.nr && cc < s.len) ? V[(long)(4 * st + kg) * s.len + cc] : 0.0;
#pragma unroll
            for (int st = 0; st < 4; ++st) x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[st], w2[st], x, 0, 0, 0);
        };
        if (TPW > 0) {
#pragma unroll
            for (int u = 0; u < TR; ++u) {
                const int tile = w + NW * u;
                if (tile >= b && tile < ntile) update_tile(tile, acc[u]);
            }
        } else {
            for (int tile = w; tile < ntile; tile += NW) {
                if (tile < b) continue;
                d4_t x;
                load(tile, x);
                update_tile(tile, x);
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const int cc = tile * WYB + 4 * rr + kg;
                    if (cc < s.len) tmp[cc] = x[rr];
                }
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

constexpr int WY_NW = 16;
constexpr int WY_MAX = WY_NW * WYB * 8;     // longest vector held in registers

}  // namespace

size_t bd_workspace(int P, int N) {
    const size_t nb = (size_t)(N + WYB - 1) / WYB;
    return (size_t)P * N + (size_t)N * P + (size_t)N * N + 2 * nb * WYB * WYB + 2 * (size_t)P + 6 * (size_t)N + 64;
}

BdWork bd_carve(double* ws, int P, int N) {
    BdWork w{};
    const size_t nb = (size_t)(N + WYB - 1) / WYB;
    w.P = P;
    w.N = N;
    w.A = ws;
    w.VQ = w.A + (size_t)P * N;
    w.VP = w.VQ + (size_t)N * P;
    w.TQ = w.VP + (size_t)N * N;
    w.TP = w.TQ + nb * WYB * WYB;
    w.col = w.TP + nb * WYB * WYB;
    w.row = w.col + P;
    w.tauq = w.row + N;
    w.taup = w.tauq + N;
    w.d = w.taup + N;
    w.e = w.d + N;
    return w;
}

void bidiagonalise(const BdWork& w, const double* theta, bool tr, hipStream_t s, LaunchProbe* probe) {
    const int P = w.P, N = w.N;
    hipLaunchKernelGGL(bd_load_kernel, dim3((N + 31) / 32, (P + 31) / 32), dim3(256), 0, s, theta, P, N, (int)tr, w.A,
                       w.col);
    for (int c = 0; c < N; ++c) {
        bool timed = probe && probe->begin(PK_BIDIAG, s);
        const int len = P - c;
        const dim3 gl(std::max(1, (N - c - 1 + 15) / 16));
        if (len > 512)
            hipLaunchKernelGGL((bd_left_kernel<1024, 32>), gl, dim3(1024), 0, s, w.A, P, N, c, w.col, w.row, w.VQ,
                               w.tauq, w.d);
        else if (len > 128)
            hipLaunchKernelGGL((bd_left_kernel<512, 16>), gl, dim3(512), 0, s, w.A, P, N, c, w.col, w.row, w.VQ,
                               w.tauq, w.d);
        else
            hipLaunchKernelGGL((bd_left_kernel<256, 8>), gl, dim3(256), 0, s, w.A, P, N, c, w.col, w.row, w.VQ,
                               w.tauq, w.d);
        if (timed) probe->end(PK_BIDIAG, s);
        if (c + 1 >= N) break;
        timed = probe && probe->begin(PK_BIDIAG, s);
        const dim3 gr((P - c - 1 + 3) / 4);
        const int cl = N - c - 1;
        if (cl > 512)
            hipLaunchKernelGGL((bd_right_kernel<32>), gr, dim3(256), 0, s, w.A, P, N, c, w.col, w.row, w.VP, w.taup,
                               w.e);
        else if (cl > 128)
            hipLaunchKernelGGL((bd_right_kernel<8>), gr, dim3(256), 0, s, w.A, P, N, c, w.col, w.row, w.VP, w.taup,
                               w.e);
        else
            hipLaunchKernelGGL((bd_right_kernel<2>), gr, dim3(256), 0, s, w.A, P, N, c, w.col, w.row, w.VP, w.taup,
                               w.e);
        if (timed) probe->end(PK_BIDIAG, s);
    }
    hipLaunchKernelGGL(wy_t_kernel, dim3((N + WYB - 1) / WYB, 2), dim3(256), 0, s, w.VQ, P, w.VP, N, w.tauq, w.taup,
                       w.TQ, w.TP);
    HIP_CHECK(hipGetLastError());
    if (probe) {
        // 4 P N^2 - 4 N^3 / 3 flops over the block read and the reflectors written
        const double p = P, n = N;
        probe->work(PK_BIDIAG, 4.0 * n * n * (p - n / 3.0), 8.0 * (2.0 * p * n + n * n));
    }
}

void bd_vectors(const BdWork& w, const double* XQ, const double* XP, const int* perm, int k, const double* sg,
                const double* scale, const BdOut& q, const BdOut& p, double* tmp, hipStream_t s, LaunchProbe* probe) {
    if (k <= 0) return;
    const int N = w.N;
    const int kr = (k + WYB - 1) / WYB * WYB;
    WySide sq{XQ, w.VQ, w.TQ, w.P, N, q.out, tmp, q.transposed, q.scaled};
    WySide sp{XP, w.VP, w.TP, N, N - 1, p.out, tmp ? tmp + (size_t)kr * w.P : nullptr, p.transposed, p.scaled};
    const dim3 grid(kr / WYB, 2);
    const bool timed = probe && probe->begin(PK_VECTORS, s);
    const int tiles = (w.P + WYB - 1) / WYB;
#define ITE_WY(NW, TPW) \
    hipLaunchKernelGGL((wy_apply_kernel<NW, TPW>), grid, dim3(64 * NW), 0, s, sq, sp, N, perm, k, sg, scale)
    if (tiles <= 4) ITE_WY(4, 1);
    else if (tiles <= 8) ITE_WY(8, 1);
    else if (tiles <= 16) ITE_WY(16, 1);
    else if (tiles <= 32) ITE_WY(16, 2);
    else if (tiles <= 64) ITE_WY(16, 4);
    else if (tiles <= WY_MAX / WYB) ITE_WY(16, 8);
    else ITE_WY(16, 0);
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
    return (size_t)((k + WYB - 1) / WYB * WYB) * ((size_t)P + N);
}

}  // namespace ite
