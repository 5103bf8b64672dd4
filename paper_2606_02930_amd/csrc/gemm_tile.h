// What the products share (matrix-core operations, parameters, the order of tiles),
// and the FP64 tile through LDS of the divide and conquer's merges (dcsvd.hip).
#pragma once

#include "internal.h"

namespace ite {
namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

constexpr int BM = 128;
constexpr int BN = 128;
constexpr int BK = 16;
constexpr int NTHREADS = 256;

template <typename T> struct MfmaOp;
template <> struct MfmaOp<double> {
    typedef d4_t acc_t;
    static constexpr int LDK = BK + 2;   // 144-byte rows: 16-byte aligned, few bank conflicts
    __device__ static acc_t mma(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // tile row of accumulator element r in lane group g = lane / 16
    __device__ static int row(int g, int r) { return 4 * r + g; }
};
template <> struct MfmaOp<float> {
    typedef f4_t acc_t;
    static constexpr int LDK = BK + 4;   // 80-byte rows
    __device__ static acc_t mma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ static int row(int g, int r) { return 4 * g + r; }
};

struct Params {
    int M, N, K;
    double alpha, beta;
    const void* A; long lda, sA;
    const void* B; long ldb, sB;
    const double* C; long ldc, sC;
    double* D; long ldd, sD;
    int mt, nt;
    float* Df;      // FP32 output instead of D (no C)
};

// Bijection from the hardware workgroup id to an output tile such that XCD x
// (workgroups with id % 8 == x) receives a contiguous range of tiles.
__device__ inline int xcd_band_tile(int bid, int T) {
    const int q = T >> 3, r = T & 7;
    const int xcd = bid & 7, idx = bid >> 3;
    const int base = xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q;
    return base + idx;
}

// D = A B for one BS x BS output tile at (m0, n0) (A M x K, B K x N, row-major; BS
// 128, 64 or 32): a K slice of 16 of each operand through LDS (As, Bs: two
// slices), four wavefronts in a 2 x 2 arrangement, each owning (BS / 2)^2 outputs
// as (BS / 32)^2 MFMA tiles of 16 x 16.  The K order of every output element
// (slices of 16, four sub-steps, lane group g supplying K index 4 g + step) does
// not depend on BS.  Ends with a barrier after the last LDS read.
template <int BS>
__device__ __forceinline__ void lds_tile(const double* __restrict__ A, long lda, const double* __restrict__ B, long ldb,
                                         double* __restrict__ D, long ldd, int M, int N, int K, int m0, int n0, double* As,
                                         double* Bs) {
    constexpr int LDK = MfmaOp<double>::LDK, IT = BS / 32, E = BS / 16;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, kg = lane >> 4;

    d4_t acc[IT][IT];
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int j = 0; j < IT; ++j) acc[i][j] = d4_t{0, 0, 0, 0};

    // a thread's share of a slice: one K index of E rows of A, E K indices of
    // one column of B
    double ra[E], rb[E];
    const int ak = t & 15, arow = t >> 4, bcol = t % BS, bk = (t / BS) * E;
    auto fetch = [&](int k0) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int row = m0 + arow + 16 * e;
            ra[e] = (row < M && k0 + ak < K) ? A[(long)row * lda + k0 + ak] : 0.0;
            const int k = k0 + bk + e;
            rb[e] = (n0 + bcol < N && k < K) ? B[(long)k * ldb + n0 + bcol] : 0.0;
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            As[(buf * BS + arow + 16 * e) * LDK + ak] = ra[e];
            Bs[(buf * BS + bcol) * LDK + bk + e] = rb[e];
        }
    };
    const int nk = (K + BK - 1) / BK;
    fetch(0);
    store(0);
    __syncthreads();

    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        const bool more = kt + 1 < nk;
        const double* Ac = As + cur * BS * LDK;
        const double* Bc = Bs + cur * BS * LDK;
        if (more) fetch((kt + 1) * BK);
        // two sub-steps of the slice at a time: 16 operand values live
        // instead of 32, which leaves room for two workgroups per CU
#pragma unroll
        for (int s2 = 0; s2 < 4; s2 += 2) {
            double a[IT][2], b[IT][2];
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const double* src = &Ac[(wm * (BS / 2) + i * 16 + l16) * LDK + 4 * kg + s2];
                a[i][0] = src[0];
                a[i][1] = src[1];
            }
#pragma unroll
            for (int j = 0; j < IT; ++j) {
                const double* src = &Bc[(wn * (BS / 2) + j * 16 + l16) * LDK + 4 * kg + s2];
                b[j][0] = src[0];
                b[j][1] = src[1];
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < IT; ++i)
#pragma unroll
                    for (int j = 0; j < IT; ++j) acc[i][j] = MfmaOp<double>::mma(a[i][s], b[j][s], acc[i][j]);
        }
        if (more) store(cur ^ 1);
        __syncthreads();
    }

    // accumulator element r of lane l holds column l % 16 and row 4 r + l / 16
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int col = n0 + wn * (BS / 2) + j * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm * (BS / 2) + i * 16 + MfmaOp<double>::row(kg, r);
                if (row < M && col < N) D[(long)row * ldd + col] = acc[i][j][r];
            }
        }
}

}  // namespace
}  // namespace ite
