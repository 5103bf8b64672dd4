// The MFMA tile of the library's FP64 and FP32 products: operand staging through
// LDS, the K loop and the epilogue of one BS x BS output tile (gemm.hip says
// how the tiles are chosen and mapped).
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

// Stage one K slice of an operand into registers (BS = 128 or 64 rows of the
// tile side, E = BS * 16 / 256 values per thread).  KC: the source is stored
// with K contiguous (rows of the tile side are strided by ld); otherwise K is
// the slow index (rows are K, the tile side is contiguous).
template <typename T, bool KC, int BS>
__device__ inline void fetch_slice(const T* __restrict__ src, long ld, int side0, int sideN, int k0,
                                   int K, int t, T (&r)[BS / 16]) {
    constexpr int E = BS / 16;
    if (KC) {
        const int kk = t & 15;
        const int k = k0 + kk;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int row = side0 + (t >> 4) + 16 * e;
            r[e] = (row < sideN && k < K) ? src[(long)row * ld + k] : T(0);
        }
    } else {
        const int col = side0 + (t % BS);
        const int kh = (t / BS) * E;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int k = k0 + kh + e;
            r[e] = (col < sideN && k < K) ? src[(long)k * ld + col] : T(0);
        }
    }
}

template <typename T, bool KC, int BS>
__device__ inline void store_slice(T* __restrict__ lds, int t, const T (&r)[BS / 16]) {
    constexpr int LDK = MfmaOp<T>::LDK, E = BS / 16;
    if (KC) {
        const int kk = t & 15;
#pragma unroll
        for (int e = 0; e < E; ++e) lds[((t >> 4) + 16 * e) * LDK + kk] = r[e];
    } else {
        const int row = t % BS;
        const int kh = (t / BS) * E;
#pragma unroll
        for (int e = 0; e < E; ++e) lds[row * LDK + kh + e] = r[e];
    }
}

// One BS x BS output tile at (m0, n0) of problem p (batch index bz): four
// wavefronts in a 2 x 2 arrangement, each owning (BS / 2)^2 outputs as
// (BS / 32)^2 MFMA tiles of 16 x 16.  The K order of every output element
// (slices of 16, four sub-steps, lane group g supplying K index 4 g + step)
// does not depend on BS, so the 128 and 64 tiles give the same bits.  As, Bs:
// LDS of two slices of each operand.  Ends with a barrier after the last LDS
// read, so the caller may start another tile.
template <typename T, bool TA, bool TB, int BS>
__device__ __forceinline__ void gemm_tile(const Params& p, int m0, int n0, long bz, T* As, T* Bs) {
    typedef typename MfmaOp<T>::acc_t acc_t;
    constexpr int LDK = MfmaOp<T>::LDK, IT = BS / 32, E = BS / 16;
    const T* __restrict__ A = static_cast<const T*>(p.A) + bz * p.sA;
    const T* __restrict__ B = static_cast<const T*>(p.B) + bz * p.sB;

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, kg = lane >> 4;

    acc_t acc[IT][IT];
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int j = 0; j < IT; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

    // A: K-contiguous unless transposed.  B: K-contiguous only when transposed.
    T ra[E], rb[E];
    const int nk = (p.K + BK - 1) / BK;
    fetch_slice<T, !TA, BS>(A, p.lda, m0, p.M, 0, p.K, t, ra);
    fetch_slice<T, TB, BS>(B, p.ldb, n0, p.N, 0, p.K, t, rb);
    store_slice<T, !TA, BS>(As, t, ra);
    store_slice<T, TB, BS>(Bs, t, rb);
    __syncthreads();

    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        const bool more = kt + 1 < nk;
        const T* Ac = As + cur * BS * LDK;
        const T* Bc = Bs + cur * BS * LDK;
        if (more) {
            fetch_slice<T, !TA, BS>(A, p.lda, m0, p.M, (kt + 1) * BK, p.K, t, ra);
            fetch_slice<T, TB, BS>(B, p.ldb, n0, p.N, (kt + 1) * BK, p.K, t, rb);
        }
        // two sub-steps of the slice at a time: 16 operand values live
        // instead of 32, which leaves room for two workgroups per CU
#pragma unroll
        for (int s2 = 0; s2 < 4; s2 += 2) {
            T a[IT][2], b[IT][2];
#pragma unroll
            for (int i = 0; i < IT; ++i) {
                const T* src = &Ac[(wm * (BS / 2) + i * 16 + l16) * LDK + 4 * kg + s2];
                a[i][0] = src[0];
                a[i][1] = src[1];
            }
#pragma unroll
            for (int j = 0; j < IT; ++j) {
                const T* src = &Bc[(wn * (BS / 2) + j * 16 + l16) * LDK + 4 * kg + s2];
                b[j][0] = src[0];
                b[j][1] = src[1];
            }
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < IT; ++i)
#pragma unroll
                    for (int j = 0; j < IT; ++j) acc[i][j] = MfmaOp<T>::mma(a[i][s], b[j][s], acc[i][j]);
        }
        if (more) {
            store_slice<T, !TA, BS>(As + (cur ^ 1) * BS * LDK, t, ra);
            store_slice<T, TB, BS>(Bs + (cur ^ 1) * BS * LDK, t, rb);
        }
        __syncthreads();
    }

    // Epilogue.  Accumulator element r of lane l holds column l % 16 of its
    // 16 x 16 tile and row 4 r + l / 16 (FP64 MFMA) or 4 (l / 16) + r (FP32).
    const double* __restrict__ C = p.C ? p.C + bz * p.sC : nullptr;
    double* __restrict__ D = p.Df ? nullptr : p.D + bz * p.sD;
    float* __restrict__ Df = p.Df ? p.Df + bz * p.sD : nullptr;
#pragma unroll
    for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int col = n0 + wn * (BS / 2) + j * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm * (BS / 2) + i * 16 + MfmaOp<T>::row(kg, r);
                if (row < p.M && col < p.N) {
                    double v = p.alpha * (double)acc[i][j][r];
                    if (Df) {
                        Df[(long)row * p.ldd + col] = (float)v;
                    } else {
                        if (C) v += p.beta * C[(long)row * p.ldc + col];
                        D[(long)row * p.ldd + col] = v;
                    }
                }
            }
        }
}

}  // namespace
}  // namespace ite
