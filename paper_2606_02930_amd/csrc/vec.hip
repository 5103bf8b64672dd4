// Bandwidth-bound kernels of the local solver: dots, norms and combinations,
// the sparse MPO contraction stage, precision conversions and small helpers.
//
// Reductions are deterministic: a fixed number of blocks (a function of n
// only), a fixed per-block order (wavefront shuffles, then LDS), and a second
// pass that sums the block partials in index order.
#include "internal.h"
#include "units.h"
#include "wave.h"

#include <cmath>
#include <stdexcept>

namespace ite {
namespace {

constexpr int RT = 256;           // threads per reduction block
constexpr int MAX_RED_BLOCKS = 512;   // two a compute unit; every block of the next launch sums them

// Block sum of v (every thread of the block gets the result).
__device__ inline double block_sum(double v, double* sh) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) sh[w] = v;
    __syncthreads();
    double r = 0.0;
    const int nw = blockDim.x >> 6;
    for (int i = 0; i < nw; ++i) r += sh[i];
    return r;
}

// Block vb of a reduction over vg blocks (the partition depends on n only,
// through vg = reduce_blocks(n)): *out = the block's share of x . y.
__device__ inline void dot_block(const double* __restrict__ x, const double* __restrict__ y, size_t n, int vb, int vg,
                                 double* __restrict__ out, double* sh) {
    double acc = 0.0;
    const size_t stride = (size_t)vg * RT;
    for (size_t i = (size_t)vb * RT + threadIdx.x; i < n; i += stride) acc += x[i] * y[i];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) *out = acc;
}

__global__ __launch_bounds__(RT) void dot_partials_kernel(const double* __restrict__ x,
                                                          const double* __restrict__ y, size_t n,
                                                          double* __restrict__ partial) {
    __shared__ double sh[RT / 64];
    dot_block(x, y, n, blockIdx.x, gridDim.x, partial + blockIdx.x, sh);
}

// *out (mode 0: =, 1: +=, 2: = sqrt) of the sum of nb partials.
__device__ inline void finish_one(const double* __restrict__ partial, int nb, double* __restrict__ out, int mode,
                                  double* sh) {
    double acc = 0.0;
    // fixed assignment of partials to threads, fixed combination order
    for (int b = threadIdx.x; b < nb; b += RT) acc += partial[b];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) {
        if (mode == 0) *out = acc;
        else if (mode == 1) *out += acc;
        else *out = sqrt(fmax(acc, 0.0));
    }
}

__global__ __launch_bounds__(RT) void finish_partials_kernel(const double* __restrict__ partial,
                                                             int nb, double* __restrict__ out,
                                                             int mode, HostPost post) {
    __shared__ double sh[RT / 64];
    const int j = blockIdx.x;
    finish_one(partial + (size_t)j * nb, nb, out + j, mode, sh);
    if (post.flag && j == 0 && threadIdx.x == 0) {
        post.data[0] = out[0];
        post_flag(post);
    }
}

template <int KMAX, bool SUB>
__global__ __launch_bounds__(RT) void gemv_kernel(const double* __restrict__ V, long ldv, int k,
                                                  const double* __restrict__ coef,
                                                  double* __restrict__ w, size_t n) {
    double c[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) c[j] = (j < k) ? coef[j] : 0.0;
    const size_t stride = (size_t)gridDim.x * RT;
    for (size_t i = (size_t)blockIdx.x * RT + threadIdx.x; i < n; i += stride) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < KMAX; ++j)
            if (j < k) s += c[j] * V[(size_t)j * ldv + i];
        w[i] = SUB ? w[i] - s : w[i] + s;
    }
}

__global__ void axpby_kernel(size_t n, double a, const double* __restrict__ x, double b,
                             const double* __restrict__ y, double* __restrict__ out) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = y ? a * x[i] + b * y[i] : a * x[i];
}

__global__ void scale_inv_kernel(const double* __restrict__ x, const double* __restrict__ den,
                                 double* __restrict__ out, size_t n) {
    const double d = *den;
    const double inv = d > 0.0 ? 1.0 / d : 0.0;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        out[i] = x[i] * inv;
}

__global__ void scale_kernel(double* __restrict__ x, double a, size_t n) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) x[i] *= a;
}

__global__ void fill_kernel(double* __restrict__ x, double v, size_t n) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) x[i] = v;
}

__global__ __launch_bounds__(1024) void max_abs_kernel(const double* __restrict__ x, size_t n, HostPost post) {
    __shared__ double sh[16];
    double m = 0.0;
    for (size_t i = threadIdx.x; i < n; i += 1024) m = isfinite(x[i]) ? fmax(m, fabs(x[i])) : INFINITY;
    m = wave_max_nonneg(m);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x > 0) return;
    for (int q = 1; q < 16; ++q) m = fmax(m, sh[q]);
    post.data[0] = m;
    post_flag(post);
}

__global__ void eye_kernel(double* __restrict__ x, int D) {
    const size_t n = (size_t)D * D;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        x[i] = (i / D == i % D) ? 1.0 : 0.0;
}

__global__ void nonfinite_kernel(const double* __restrict__ x, size_t n, int* flag) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        bad |= !isfinite(x[i]);
    if (bad) atomicOr(flag, 1);
}

__global__ void f32_kernel(const double* __restrict__ x, float* __restrict__ y, size_t n) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        y[i] = (float)x[i];
}

// FP64 -> BF16 with round to nearest even, done in two exact steps: the FP64
// value is first rounded to FP32 with round-to-odd (so that the second
// rounding cannot double-round), then FP32 -> BF16 by the usual
// add-0x7fff-plus-lsb rule.  NaN stays NaN.
__device__ inline uint16_t to_bf16(double v) {
    float f = (float)v;
    if (isfinite(f) && (double)f != v) {
        // round to odd: truncate toward zero, then set the last bit
        uint32_t u = __float_as_uint(f);
        if (fabs((double)f) > fabs(v)) u -= 1;   // move toward zero
        u |= 1u;
        f = __uint_as_float(u);
    }
    uint32_t u = __float_as_uint(f);
    if (isnan(f)) return (uint16_t)((u >> 16) | 0x40);
    const uint32_t lsb = (u >> 16) & 1u;
    u += 0x7fffu + lsb;
    return (uint16_t)(u >> 16);
}

__global__ void bf16_kernel(const double* __restrict__ x, uint16_t* __restrict__ y, size_t n) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        y[i] = to_bf16(x[i]);
}

// out[j][i] = in[i][j] through a 32 x 32 LDS tile.
__global__ void transpose_kernel(const double* __restrict__ in, int rows, int cols,
                                 double* __restrict__ out) {
    __shared__ double tile[32][33];
    const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
    for (int k = threadIdx.y; k < 32; k += blockDim.y) {
        const int r = r0 + k, c = c0 + threadIdx.x;
        if (r < rows && c < cols) tile[k][threadIdx.x] = in[(size_t)r * cols + c];
    }
    __syncthreads();
    for (int k = threadIdx.y; k < 32; k += blockDim.y) {
        const int c = c0 + k, r = r0 + threadIdx.x;
        if (r < rows && c < cols) out[(size_t)c * rows + r] = tile[threadIdx.x][k];
    }
}

// ---------------------------------------------------------------------------
// Sparse MPO stage.  A workgroup handles one g and CL V consecutive columns
// (CL = 2^lc lanes of V columns): the I inputs of those columns and the CSR
// matrix are staged in LDS, then the STAGE_NT / CL groups of lanes share the O
// outputs.  It is a copy with a few multiply-adds, so memory bounds it when
// it is large and latency when it is small: the lanes over the outputs keep
// the chain of LDS reads short and let a small column tile fill the chip
// without idle lanes.  Against one thread a column looping over all outputs,
// whose inputs left room for one or two wavefronts a compute unit: bond 32
// (d 2, w 5) 13.4 -> 3.7 us, bond 64 (d 4, w 6) 62 -> 4.7, bond 1024 (d 2)
// 121 -> 59 us (5.7 TB/s), FP32 in and BF16 out at bond 256 (d 4) 87 -> 16.  The terms of an output are summed in CSR order
// whatever the tile.
// V = 4: unit column strides, every stride a multiple of 4, 16-byte aligned
// bases: 16-byte loads and stores.  V = 1: any strides.
// OUT: 0 writes FP64 to st.out, 1 rounds to FP32 and 2 to BF16 into st.out_lo
// (the operand of a following low-precision contraction).
// ---------------------------------------------------------------------------
constexpr int STAGE_NT = 256;
constexpr size_t STAGE_LDS = 128 * 1024;
// LDS of a stage workgroup: the inputs (at most STAGE_LDS) and, when it fits,
// the CSR matrix behind them
constexpr size_t STAGE_LDS_TOTAL = 152 * 1024;

template <int V, typename TIN>
__device__ inline void load_cols(const TIN* p, TIN (&v)[V]) {
    if constexpr (V == 1) {
        v[0] = p[0];
    } else if constexpr (sizeof(TIN) == 4) {
        const float4 q = *reinterpret_cast<const float4*>(p);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
        const double2 a = *reinterpret_cast<const double2*>(p);
        const double2 b = *reinterpret_cast<const double2*>(p + 2);
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    }
}

// Columns cb .. cb + CL V - 1 of group g; xin: LDS of I CL V inputs of type
// TIN ([I][V][CL]: lane-contiguous reads), then the CSR copy.
template <int OUT, int V, typename TIN>
__device__ inline void stage_tile(const Stage& st, int g, int cb, int lc, TIN* xin) {
    const int CL = 1 << lc, OG = STAGE_NT >> lc;
    const int t = threadIdx.x, cl = t & (CL - 1), og = t >> lc;
    const int c = cb + cl * V;
    const bool live = c < st.C;
    const TIN* __restrict__ in;
    if constexpr (sizeof(TIN) == 4) in = st.in_f32;
    else in = st.in;
    in += (long)g * st.in_gs + (long)c * (V == 1 ? st.in_cs : 1);
    const bool in_flat = st.in_div == 1;   // no division in the common layout
    for (int i = og; i < st.I; i += OG) {
        TIN v[V];
#pragma unroll
        for (int q = 0; q < V; ++q) v[q] = 0;
        const long off = in_flat ? (long)i * st.in_s1
                                 : (long)(i / st.in_div) * st.in_s1 + (long)(i % st.in_div) * st.in_s2;
        if (live) load_cols<V>(in + off, v);
#pragma unroll
        for (int q = 0; q < V; ++q) xin[(i * V + q) * CL + cl] = v[q];
    }
    // the CSR matrix in LDS when it fits behind the inputs (read as
    // broadcasts instead of a chain of dependent scalar loads)
    const int nnz = st.nnz;
    const bool lcsr = st.csr_lds != 0;
    double* sval = reinterpret_cast<double*>(xin + ((size_t)st.I * V << lc));
    int* scol = reinterpret_cast<int*>(sval + nnz);
    int* srow = scol + nnz;
    if (lcsr) {
        for (int e = t; e < nnz; e += STAGE_NT) {
            sval[e] = st.val[e];
            scol[e] = st.col[e];
        }
        for (int o = t; o <= st.O; o += STAGE_NT) srow[o] = st.rowptr[o];
    }
    __syncthreads();
    if (live) {
        const int* rp = lcsr ? srow : st.rowptr;
        const int* col = lcsr ? scol : st.col;
        const double* val = lcsr ? sval : st.val;
        const long base = (long)g * st.out_gs + (long)c * (V == 1 ? st.out_cs : 1);
        const bool out_flat = st.out_div == 1;
        for (int o = og; o < st.O; o += OG) {
            double acc[V];
#pragma unroll
            for (int q = 0; q < V; ++q) acc[q] = 0.0;
            const int e1 = rp[o + 1];
            for (int e = rp[o]; e < e1; ++e) {
                const double w = val[e];
                const TIN* x = xin + ((col[e] * V) << lc) + cl;
#pragma unroll
                for (int q = 0; q < V; ++q) acc[q] += w * (double)x[q << lc];
            }
            const long at = base + (out_flat ? (long)o * st.out_s1
                                             : (long)(o / st.out_div) * st.out_s1 + (long)(o % st.out_div) * st.out_s2);
            if constexpr (OUT == 0) {
                if constexpr (V == 1) {
                    st.out[at] = acc[0];
                } else {
                    *reinterpret_cast<double2*>(st.out + at) = double2{acc[0], acc[1]};
                    *reinterpret_cast<double2*>(st.out + at + 2) = double2{acc[2], acc[3]};
                }
            } else if constexpr (OUT == 1) {
                float* out = static_cast<float*>(st.out_lo) + at;
                if constexpr (V == 1) *out = (float)acc[0];
                else *reinterpret_cast<float4*>(out) = float4{(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
            } else {
                uint16_t* out = static_cast<uint16_t*>(st.out_lo) + at;
                if constexpr (V == 1) {
                    *out = to_bf16(acc[0]);
                } else {
                    uint2 v;
                    v.x = (uint32_t)to_bf16(acc[0]) | ((uint32_t)to_bf16(acc[1]) << 16);
                    v.y = (uint32_t)to_bf16(acc[2]) | ((uint32_t)to_bf16(acc[3]) << 16);
                    *reinterpret_cast<uint2*>(out) = v;
                }
            }
        }
    }
}

template <int OUT, int V, typename TIN>
__global__ __launch_bounds__(STAGE_NT) void stage_kernel(Stage st, int lc) {
    extern __shared__ double stage_lds[];
    stage_tile<OUT, V, TIN>(st, blockIdx.y, (blockIdx.x * V) << lc, lc, reinterpret_cast<TIN*>(stage_lds));
}

inline int grid_for(size_t n, int threads, int cap = 4096) {
    size_t b = (n + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > (size_t)cap) b = cap;
    return (int)b;
}

}  // namespace

int reduce_blocks(size_t n) {
    size_t b = (n + RT * 4 - 1) / (RT * 4);
    if (b < 1) b = 1;
    if (b > MAX_RED_BLOCKS) b = MAX_RED_BLOCKS;
    return (int)b;
}

void dot_partials(const double* x, const double* y, size_t n, double* partial, hipStream_t s) {
    hipLaunchKernelGGL(dot_partials_kernel, dim3(reduce_blocks(n)), dim3(RT), 0, s, x, y, n, partial);
    HIP_CHECK(hipGetLastError());
}

void finish_partials(const double* partial, int k, int nb, double* out, int mode, hipStream_t s,
                     HostPost post) {
    hipLaunchKernelGGL(finish_partials_kernel, dim3(k), dim3(RT), 0, s, partial, nb, out, mode, post);
    HIP_CHECK(hipGetLastError());
}

template <bool SUB>
static void gemv_launch(const double* V, long ldv, int k, const double* coef, double* w, size_t n,
                        hipStream_t s) {
    const int nb = grid_for(n, RT);
    for (int j0 = 0; j0 < k; j0 += 16) {
        const int kk = k - j0 < 16 ? k - j0 : 16;
        if (kk <= 4)
            hipLaunchKernelGGL((gemv_kernel<4, SUB>), dim3(nb), dim3(RT), 0, s, V + (size_t)j0 * ldv, ldv, kk,
                               coef + j0, w, n);
        else if (kk <= 8)
            hipLaunchKernelGGL((gemv_kernel<8, SUB>), dim3(nb), dim3(RT), 0, s, V + (size_t)j0 * ldv, ldv, kk,
                               coef + j0, w, n);
        else
            hipLaunchKernelGGL((gemv_kernel<16, SUB>), dim3(nb), dim3(RT), 0, s, V + (size_t)j0 * ldv, ldv, kk,
                               coef + j0, w, n);
    }
    HIP_CHECK(hipGetLastError());
}

void gemv_sub(const double* V, long ldv, int k, const double* coef, double* w, size_t n, hipStream_t s) {
    gemv_launch<true>(V, ldv, k, coef, w, n, s);
}
void gemv_add(const double* V, long ldv, int k, const double* coef, double* x, size_t n, hipStream_t s) {
    gemv_launch<false>(V, ldv, k, coef, x, n, s);
}

void axpby(size_t n, double a, const double* x, double b, const double* y, double* out, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(axpby_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, n, a, x, b, y, out);
    HIP_CHECK(hipGetLastError());
}

// One site of the conditional sampling of an MPS in the product basis, one
// workgroup per sample: T[smp] ([d][Dr]) = v A_site for that sample's
// normalised left vector v; p_s = ||T[smp][s]||^2 (fixed reduction order);
// the site takes the first s with p_0 + .. + p_s > u[smp] (p_0 + .. + p_(d-1))
// and p_s > 0 (else the last s with p_s > 0, else 0), written to
// cfg[smp * L + site]; vnext[smp] = T[smp][s] / ||T[smp][s]||.  A total that
// is zero or not finite (a zero or non-finite state) sets flag[0] = 1, a
// uniform outside [0, 1) flag[1] = 1.
constexpr int SMP_T = 256;
__global__ __launch_bounds__(SMP_T) void sample_site_kernel(const double* __restrict__ T, int d, int Dr,
                                                            const double* __restrict__ u,
                                                            double* __restrict__ vnext, int* __restrict__ cfg,
                                                            int L, int site, double* __restrict__ flag) {
    __shared__ double part[SMP_T / 64][SAMPLE_DMAX];
    __shared__ double pw[SAMPLE_DMAX];
    __shared__ int chosen;
    const int smp = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const double* row = T + (size_t)smp * d * Dr;
    for (int q = 0; q < d; ++q) {
        double acc = 0.0;
        for (int j = t; j < Dr; j += SMP_T) {
            const double x = row[(size_t)q * Dr + j];
            acc += x * x;
        }
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);   // butterfly: fixed order
        if (lane == 0) part[wv][q] = acc;
    }
    __syncthreads();
    if (t == 0) {
        double tot = 0.0;
        for (int q = 0; q < d; ++q) {
            double pq = 0.0;
            for (int w = 0; w < SMP_T / 64; ++w) pq += part[w][q];
            pw[q] = pq;
            tot += pq;
        }
        if (!(tot > 0.0) || !isfinite(tot)) flag[0] = 1.0;
        if (!(u[smp] >= 0.0 && u[smp] < 1.0)) flag[1] = 1.0;
        const double thr = u[smp] * tot;
        int pick = -1;
        double cum = 0.0;
        for (int q = 0; q < d; ++q) {
            cum += pw[q];
            if (pick < 0 && cum > thr && pw[q] > 0.0) pick = q;
        }
        for (int q = d - 1; q >= 0 && pick < 0; --q)
            if (pw[q] > 0.0) pick = q;
        if (pick < 0) pick = 0;
        chosen = pick;
        cfg[(size_t)smp * L + site] = pick;
    }
    __syncthreads();
    const int q = chosen;
    const double nq = pw[q];
    const double inv = nq > 0.0 ? 1.0 / sqrt(nq) : 0.0;
    for (int j = t; j < Dr; j += SMP_T) vnext[(size_t)smp * Dr + j] = row[(size_t)q * Dr + j] * inv;
}

void sample_site(const double* T, int nsamples, int d, int Dr, const double* u, double* vnext, int* cfg, int L,
                 int site, double* flag, hipStream_t s) {
    if (nsamples <= 0) return;
    if (d < 1 || d > SAMPLE_DMAX || Dr < 1) throw std::invalid_argument("sample_site: bad dimensions");
    hipLaunchKernelGGL(sample_site_kernel, dim3(nsamples), dim3(SMP_T), 0, s, T, d, Dr, u, vnext, cfg, L, site,
                       flag);
    HIP_CHECK(hipGetLastError());
}

void scale_inv(const double* x, const double* den, double* out, size_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(scale_inv_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, den, out, n);
    HIP_CHECK(hipGetLastError());
}

// Lowest eigenpair of the Lanczos cycle's projected matrix, on the device
// (one wavefront): T (kused x kused, symmetric) from the Gram-Schmidt
// coefficients of the columns hd[k * HESS_HC ..] (both passes summed, the
// upper triangle mirrored), kused the steps up to the first breakdown (a
// next norm <= 1e-14 of the largest diagonal so far); cyclic Jacobi rotations
// (each zeroes t_pq with tan the smaller root of t^2 + 2 tau t - 1 = 0,
// tau = (t_qq - t_pp) / (2 t_pq)) until the off-diagonal mass is below 1e-32
// of the total (at most 60 sweeps); y = the eigenvector of the smallest
// eigenvalue (zero beyond kused).  rec: [0] the eigenvalue, [1] the residual
// estimate |h_(k+1,k) y_k| / |theta| (its absolute value when theta = 0),
// [2] += kused, [3] kused.
__global__ __launch_bounds__(64) void lanczos_eig_kernel(const double* __restrict__ hd, int mm,
                                                         double* __restrict__ y, double* __restrict__ rec) {
    __shared__ double A[HESS_KMAX][HESS_KMAX + 1];
    __shared__ double Z[HESS_KMAX][HESS_KMAX + 1];
    __shared__ double cs[2];
    __shared__ int ku;
    __shared__ double red[2];
    const int t = threadIdx.x;
    if (t == 0) {
        int kused = mm;
        double scale_h = 0.0;
        for (int k = 0; k < mm; ++k) {
            const double* col = hd + (size_t)k * HESS_HC;
            scale_h = fmax(scale_h, fabs(col[k] + col[64 + k]));
            if (k + 1 < mm && !(col[128] > 1e-14 * fmax(scale_h, 1e-300))) {
                kused = k + 1;
                break;
            }
        }
        ku = kused;
    }
    __syncthreads();
    const int k = ku;
    for (int c = 0; c < k; ++c) {
        const double* col = hd + (size_t)c * HESS_HC;
        if (t <= c) {
            const double v = col[t] + col[64 + t];
            A[t][c] = v;
            A[c][t] = v;
        }
        if (t < k) Z[c][t] = c == t ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int sweep = 0; sweep < 60; ++sweep) {
        if (t == 0) {
            double off = 0.0, tot = 0.0;
            for (int i = 0; i < k; ++i)
                for (int j = 0; j < k; ++j) {
                    const double v = A[i][j] * A[i][j];
                    tot += v;
                    if (i != j) off += v;
                }
            red[0] = off;
            red[1] = tot;
        }
        __syncthreads();
        if (!(red[0] > 1e-32 * red[1])) break;
        for (int p = 0; p < k; ++p)
            for (int q = p + 1; q < k; ++q) {
                if (t == 0) {
                    const double apq = A[p][q];
                    double cc = 1.0, ss = 0.0;
                    if (apq != 0.0) {
                        const double tau = (A[q][q] - A[p][p]) / (2.0 * apq);
                        const double tt = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                        cc = 1.0 / sqrt(1.0 + tt * tt);
                        ss = tt * cc;
                    }
                    cs[0] = cc;
                    cs[1] = ss;
                }
                __syncthreads();
                const double cc = cs[0], ss = cs[1];
                if (ss != 0.0) {
                    if (t < k) {   // columns p, q of A J
                        const double arp = A[t][p], arq = A[t][q];
                        A[t][p] = cc * arp - ss * arq;
                        A[t][q] = ss * arp + cc * arq;
                    }
                    __syncthreads();
                    if (t < k) {   // rows p, q of J^T (A J); Z J
                        const double apr = A[p][t], aqr = A[q][t];
                        A[p][t] = cc * apr - ss * aqr;
                        A[q][t] = ss * apr + cc * aqr;
                        const double zrp = Z[t][p], zrq = Z[t][q];
                        Z[t][p] = cc * zrp - ss * zrq;
                        Z[t][q] = ss * zrp + cc * zrq;
                    }
                }
                __syncthreads();
            }
    }
    if (t == 0) {
        int imin = 0;
        for (int i = 1; i < k; ++i)
            if (A[i][i] < A[imin][imin]) imin = i;
        red[0] = imin;
        const double theta = A[imin][imin];
        const double hlast = k == mm ? hd[(size_t)(mm - 1) * HESS_HC + 128] : 0.0;
        const double res = fabs(hlast * Z[k - 1][imin]);
        rec[0] = theta;
        rec[1] = theta != 0.0 ? res / fabs(theta) : res;
        rec[2] += k;
        rec[3] = k;
    }
    __syncthreads();
    const int imin = (int)red[0];
    if (t < mm) y[t] = t < k ? Z[t][imin] : 0.0;
}

void lanczos_eig(const double* hd, int mm, double* y, double* rec, hipStream_t s) {
    if (mm < 1 || mm > HESS_KMAX) ITE_FAIL(ITE_EINVAL, "lanczos_eig: Krylov dimension outside 1..64");
    hipLaunchKernelGGL(lanczos_eig_kernel, dim3(1), dim3(64), 0, s, hd, mm, y, rec);
    HIP_CHECK(hipGetLastError());
}

void scale(double* x, double a, size_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(scale_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, a, n);
    HIP_CHECK(hipGetLastError());
}

void max_abs(const double* x, size_t n, const HostPost& post, hipStream_t s) {
    hipLaunchKernelGGL(max_abs_kernel, dim3(1), dim3(1024), 0, s, x, n, post);
    HIP_CHECK(hipGetLastError());
}

void fill(double* x, double v, size_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, v, n);
    HIP_CHECK(hipGetLastError());
}

void eye(double* x, int D, hipStream_t s) {
    hipLaunchKernelGGL(eye_kernel, dim3(grid_for((size_t)D * D, 256)), dim3(256), 0, s, x, D);
    HIP_CHECK(hipGetLastError());
}

void nonfinite_any(const double* x, size_t n, int* flag, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(nonfinite_kernel, dim3(grid_for(n, 256, 1024)), dim3(256), 0, s, x, n, flag);
    HIP_CHECK(hipGetLastError());
}

void convert_f32(const double* x, float* y, size_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(f32_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, y, n);
    HIP_CHECK(hipGetLastError());
}

void convert_bf16(const double* x, uint16_t* y, size_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(bf16_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, x, y, n);
    HIP_CHECK(hipGetLastError());
}

void transpose(const double* in, int rows, int cols, double* out, hipStream_t s) {
    if (rows <= 0 || cols <= 0) return;
    dim3 grid((cols + 31) / 32, (rows + 31) / 32);
    hipLaunchKernelGGL(transpose_kernel, grid, dim3(32, 8), 0, s, in, rows, cols, out);
    HIP_CHECK(hipGetLastError());
}

// Whether the four-column kernel applies: unit column strides, strides and
// the column count multiples of 4, 16-byte aligned bases.
static bool stage4_ok(const Stage& st) {
    auto m4 = [](long v) { return v % 4 == 0; };
    auto al = [](const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; };
    if (st.in_cs != 1 || st.out_cs != 1 || st.C % 4 != 0) return false;
    if (!m4(st.in_gs) || !m4(st.in_s1) || (st.in_div > 1 && !m4(st.in_s2))) return false;
    if (!m4(st.out_gs) || !m4(st.out_s1) || (st.out_div > 1 && !m4(st.out_s2))) return false;
    const void* in = st.in_f32 ? static_cast<const void*>(st.in_f32) : static_cast<const void*>(st.in);
    if (!al(in, 16)) return false;
    if (st.out_prec == 0) return al(st.out, 16);
    return al(st.out_lo, st.out_prec == 1 ? 16 : 8);
}

// Column tile: as wide as leaves four workgroups a compute unit and their
// inputs in a quarter of its LDS, but 16 columns (a 128-byte line of FP64) at
// least; the narrowest tile holds the 1024 inputs of the largest stage an MPO
// can have (w = 16, d = 8) in STAGE_LDS.
template <int V, typename TIN>
static void stage_launch(Stage st, hipStream_t s) {
    constexpr int LMIN = V == 4 ? 2 : 4;
    int lc = 6;
    auto blocks = [&] { return (long)st.G * ((st.C + (V << lc) - 1) / (V << lc)); };
    while (lc > LMIN && (blocks() < 1024 || ((size_t)st.I * V * sizeof(TIN) << lc) > 36 * 1024)) --lc;
    const dim3 grid((st.C + (V << lc) - 1) / (V << lc), st.G);
    size_t lds = (size_t)st.I * V * sizeof(TIN) << lc;
    const size_t csr = (size_t)st.nnz * 12 + (size_t)(st.O + 1) * 4;
    st.csr_lds = st.nnz >= 0 && lds + csr <= STAGE_LDS_TOTAL;
    if (st.csr_lds) lds += csr;
    if (st.out_prec == 0) hipLaunchKernelGGL((stage_kernel<0, V, TIN>), grid, dim3(STAGE_NT), lds, s, st, lc);
    else if (st.out_prec == 1) hipLaunchKernelGGL((stage_kernel<1, V, TIN>), grid, dim3(STAGE_NT), lds, s, st, lc);
    else hipLaunchKernelGGL((stage_kernel<2, V, TIN>), grid, dim3(STAGE_NT), lds, s, st, lc);
    HIP_CHECK(hipGetLastError());
}

void stage_f64(const Stage& st, hipStream_t s) {
    if (st.G <= 0 || st.C <= 0 || st.O <= 0) return;
    if (st.I < 1 || (size_t)st.I * 16 * sizeof(double) > STAGE_LDS)
        ITE_FAIL(ITE_EINVAL, "MPO stage: more than 1024 inputs per column");
    if (stage4_ok(st)) {
        if (st.in_f32) stage_launch<4, float>(st, s);
        else stage_launch<4, double>(st, s);
    } else {
        if (st.in_f32) stage_launch<1, float>(st, s);
        else stage_launch<1, double>(st, s);
    }
}

// ---------------------------------------------------------------------------
// Batched fixed-budget GMRES (see BatchVec in internal.h)
// ---------------------------------------------------------------------------
namespace {

// x += sum_j c_j V_j at entry i, in chunks of 16 basis vectors as gemv_launch does.
__device__ inline double gemv_elem(const double* __restrict__ V, long ldv, int k, const double* __restrict__ c,
                                   double x, size_t i) {
    for (int j0 = 0; j0 < k; j0 += 16) {
        const int kk = k - j0 < 16 ? k - j0 : 16;
        double s = 0.0;
        for (int j = 0; j < kk; ++j) s += c[j0 + j] * V[(size_t)(j0 + j) * ldv + i];
        x += s;
    }
    return x;
}

__global__ __launch_bounds__(RT) void batch_vec_kernel(const BatchVec* __restrict__ d, int G,
                                                       const int* __restrict__ tot, int op, int k) {
    const int total = tot[BT_EW];
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int g = unit_problem(u, G, [&](int q) { return d[q].ew_start; });
        const BatchVec& p = d[g];
        const size_t i0 = (size_t)(u - p.ew_start) * BATCH_EW;
        const size_t i1 = min((size_t)p.n, i0 + BATCH_EW);
        if (op == 0) {
            for (size_t i = i0 + threadIdx.x; i < i1; i += RT) p.x[i] = gemv_elem(p.V, p.n, k, p.y, p.x[i], i);
        } else {
            const double* vk = p.V + (size_t)k * p.n;
            for (size_t i = i0 + threadIdx.x; i < i1; i += RT) p.tlo[i] = (float)vk[i];
        }
    }
}

// LO: the FP32 stage st_lo (FP32 output) instead of st.
template <bool LO>
__global__ __launch_bounds__(STAGE_NT) void batch_stage_kernel(const BatchVec* __restrict__ d, int G,
                                                               const int* __restrict__ tot) {
    __shared__ double lds[(BATCH_STAGE_I << BATCH_STAGE_LC) + BATCH_STAGE_CSR / 8];
    const int total = tot[LO ? BT_STAGE_LO : BT_STAGE];
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int g = unit_problem(u, G, [&](int q) { return LO ? d[q].stage_lo_start : d[q].stage_start; });
        const Stage& st = LO ? d[g].st_lo : d[g].st;
        const int nc = (st.C + (1 << BATCH_STAGE_LC) - 1) >> BATCH_STAGE_LC;
        const int lu = u - (LO ? d[g].stage_lo_start : d[g].stage_start);
        const int cb = (lu % nc) << BATCH_STAGE_LC;
        if (LO) stage_tile<1, 1, float>(st, lu / nc, cb, BATCH_STAGE_LC, reinterpret_cast<float*>(lds));
        else stage_tile<0, 1, double>(st, lu / nc, cb, BATCH_STAGE_LC, lds);
        __syncthreads();   // the LDS is the next unit's
    }
}

}  // namespace

void batch_vec(const BatchVec* d, int G, const int* tot, int op, int k, hipStream_t s) {
    if (G <= 0) return;
    hipLaunchKernelGGL(batch_vec_kernel, dim3(BATCH_GRID), dim3(RT), 0, s, d, G, tot, op, k);
    HIP_CHECK(hipGetLastError());
}

void batch_stage(const BatchVec* d, int G, const int* tot, hipStream_t s) {
    if (G <= 0) return;
    hipLaunchKernelGGL(batch_stage_kernel<false>, dim3(BATCH_GRID), dim3(STAGE_NT), 0, s, d, G, tot);
    HIP_CHECK(hipGetLastError());
}

void batch_stage_lo(const BatchVec* d, int G, const int* tot, hipStream_t s) {
    if (G <= 0) return;
    hipLaunchKernelGGL(batch_stage_kernel<true>, dim3(BATCH_GRID), dim3(STAGE_NT), 0, s, d, G, tot);
    HIP_CHECK(hipGetLastError());
}

}  // namespace ite
