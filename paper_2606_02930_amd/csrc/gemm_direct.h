// Products whose operands go from memory straight into the matrix-core
// registers (gemm.hip says when a product is done this way).
#pragma once

#include "gemm_tile.h"

namespace ite {
namespace {

// N values of T at any element alignment, one load instruction per 16 bytes.
template <typename T, int N> struct ElemVec {
    typedef T type __attribute__((ext_vector_type(N), aligned(sizeof(T))));
};
template <typename T> struct ElemVec<T, 1> { typedef T type; };

template <typename T, int N>
__device__ inline void load_elems(const T* __restrict__ src, T (&v)[N]) {
    if constexpr (N == 1) v[0] = src[0];
    else {
        const typename ElemVec<T, N>::type x = *reinterpret_cast<const typename ElemVec<T, N>::type*>(src);
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = x[i];
    }
}

// One operand of a wavefront's 16 S-wide tile side: the values of a K slice
// of 16 as v[tile][step], lane group g = lane / 16 supplying K index
// 4 g + step.  `load` fetches a slice into registers,
// `values` turns it into v.
//
// KC: K is the contiguous index.  A lane's values are four of one row, so
// lanes read straight from memory would touch 16 cache lines with every
// quarter wavefront; the slice is fetched with consecutive lanes along a row
// instead and passes through a piece of LDS of the wavefront's own (rows of
// LDK, no barrier).  Otherwise the side is contiguous and a lane reads S
// neighbours of its four K rows, so tile t holds the side's indices S l + t.
//
// Indices past the end of the side are clamped or cannot occur (the caller
// places a side-contiguous tile of S > 1 inside the side): what they give is
// not stored.
template <typename T, bool KC, int S> struct Side;

template <typename T, int S> struct Side<T, true, S> {
    static constexpr int EV = 16 / (int)sizeof(T);       // values of a 16-byte load
    static constexpr int CH = BK / EV;                   // loads of a row
    static constexpr int NL = 16 * S * CH / 64;          // loads of a lane
    static constexpr int LDK = MfmaOp<T>::LDK;
    static constexpr int LDS = 16 * S * LDK;
    struct Slice { T v[NL][EV]; };
    const T* ptr[NL];
    T* lds;
    int lane;
    __device__ void init(const T* src, long ld, int side0, int sideN, int lane_, T* lds_) {
        lane = lane_;
        lds = lds_;
#pragma unroll
        for (int n = 0; n < NL; ++n)
            ptr[n] = src + (long)min(side0 + n * (64 / CH) + lane / CH, sideN - 1) * ld + (lane % CH) * EV;
    }
    // index within the side of position `pos` of tile t
    __device__ static int index(int t, int pos) { return 16 * t + pos; }
    __device__ void load(int k0, Slice& r) const {
#pragma unroll
        for (int n = 0; n < NL; ++n) load_elems<T, EV>(ptr[n] + k0, r.v[n]);
    }
    // the last, partial slice: zeros from K on
    __device__ void load_tail(int k0, int K, Slice& r) const {
#pragma unroll
        for (int n = 0; n < NL; ++n)
#pragma unroll
            for (int e = 0; e < EV; ++e)
                r.v[n][e] = k0 + (lane % CH) * EV + e < K ? ptr[n][k0 + e] : T(0);
    }
    __device__ void values(const Slice& r, T (&v)[S][4]) const {
        typedef T vec_t __attribute__((ext_vector_type(EV)));
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            vec_t x;
#pragma unroll
            for (int e = 0; e < EV; ++e) x[e] = r.v[n][e];
            *reinterpret_cast<vec_t*>(&lds[(n * (64 / CH) + lane / CH) * LDK + (lane % CH) * EV]) = x;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
            for (int h = 0; h < 4; h += EV) {
                const vec_t x = *reinterpret_cast<const vec_t*>(&lds[(16 * i + (lane & 15)) * LDK + 4 * (lane >> 4) + h]);
#pragma unroll
                for (int e = 0; e < EV; ++e) v[i][h + e] = x[e];
            }
    }
};

template <typename T, int S> struct Side<T, false, S> {
    static constexpr int LDS = 0;
    struct Slice { T v[4][S]; };
    const T* ptr;
    long ld;
    int kg;
    __device__ void init(const T* src, long ld_, int side0, int sideN, int lane, T*) {
        ld = ld_;
        kg = lane >> 4;
        const int l16 = lane & 15;
        ptr = src + (S == 1 ? min(side0 + l16, sideN - 1) : side0 + S * l16) + (long)(4 * kg) * ld;
    }
    __device__ static int index(int t, int pos) { return S * pos + t; }
    __device__ void load(int k0, Slice& r) const {
#pragma unroll
        for (int s = 0; s < 4; ++s) load_elems<T, S>(ptr + (long)(k0 + s) * ld, r.v[s]);
    }
    __device__ void load_tail(int k0, int K, Slice& r) const {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < S; ++i) r.v[s][i] = k0 + 4 * kg + s < K ? ptr[(long)(k0 + s) * ld + i] : T(0);
    }
    __device__ void values(const Slice& r, T (&v)[S][4]) const {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < S; ++i) v[i][s] = r.v[s][i];
    }
};

// The end of a tile: the K parts summed in order and in FP64 through LDS (KS
// parts of WM WN MI NI 256 values; unused for one part), alpha, beta and the
// store of the rows and columns from (ms, ns) on that are inside.  row(i, r),
// col(j): the matrix row and column of this lane's accumulator element r of
// tile (i, j).  out: nothing of the wavefront's tile is inside.
template <int MI, int NI, int WM, int WN, int KS, typename T, typename Acc, typename Row, typename Col>
__device__ __forceinline__ void finish_tile(const Params& p, long bz, int ms, int ns, bool out,
                                            const Acc (&acc)[MI][NI], Row row, Col col, T* lds) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = wave / (WM * WN), wmn = wave % (WM * WN);
    const double* C = p.C ? p.C + bz * p.sC : nullptr;
    double* D = p.Df ? nullptr : p.D + bz * p.sD;
    float* Df = p.Df ? p.Df + bz * p.sD : nullptr;
    auto store = [&](int i, int j, int r, double sum) {
        const int m = row(i, r), n = col(j);
        if (m >= ms && m < p.M && n >= ns && n < p.N) {
            double v = p.alpha * sum;
            if (Df) {
                Df[(long)m * p.ldd + n] = (float)v;
            } else {
                if (C) v += p.beta * C[(long)m * p.ldc + n];
                D[(long)m * p.ldd + n] = v;
            }
        }
    };
    if constexpr (KS == 1) {
        if (out) return;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) store(i, j, r, (double)acc[i][j][r]);
    } else {
        constexpr int E = MI * NI * 4;               // values of a lane
        constexpr int PART = WM * WN * E * 64;
        __syncthreads();
        T* mine = lds + ks * PART + wmn * E * 64 + lane;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) mine[((i * NI + j) * 4 + r) * 64] = acc[i][j][r];
        __syncthreads();
        if (!out) {
            const T* sum0 = lds + wmn * E * 64 + lane;
            // values ks, ks + KS, ... of this wavefront's tile
#pragma unroll
            for (int e0 = 0; e0 < E; e0 += KS) {
                const int e = e0 + ks;
                if (E % KS == 0 || e < E) {
                    double v = (double)sum0[e * 64];
#pragma unroll
                    for (int q = 1; q < KS; ++q) v += (double)sum0[q * PART + e * 64];
                    store(e / (4 * NI), (e / 4) % NI, e % 4, v);
                }
            }
        }
    }
}

// A (16 MI WM) x (16 NI WN) output tile at (m0, n0): WM x WN wavefronts of
// MI x NI matrix-core tiles, and KS such groups that take a part of the K
// slices each; the parts are summed in order and in FP64 through LDS (lds:
// direct_lds values).  PD slices are in flight per wavefront.  A side of more than one tile per wavefront that is
// side-contiguous (A transposed, B not) must be at least 16 MI (16 NI) long.
template <typename T, bool TA, bool TB, int MI, int NI, int WM, int WN, int KS>
constexpr int direct_lds() {
    constexpr int stage = WM * WN * KS * (Side<T, !TA, MI>::LDS + Side<T, TB, NI>::LDS);
    constexpr int parts = KS == 1 ? 1 : KS * WM * WN * MI * NI * 256;
    return stage > parts ? stage : parts;
}

template <typename T, bool TA, bool TB, int MI, int NI, int WM, int WN, int KS, int PD>
__device__ __forceinline__ void direct_tile(const Params& p, int m0, int n0, long bz, T* lds) {
    typedef typename MfmaOp<T>::acc_t acc_t;
    const T* __restrict__ A = static_cast<const T*>(p.A) + bz * p.sA;
    const T* __restrict__ B = static_cast<const T*>(p.B) + bz * p.sB;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = wave / (WM * WN), wmn = wave % (WM * WN);
    // first row and column to store, and those of the tile, moved back into
    // the side where it would end outside
    const int ms = m0 + (wmn / WN) * 16 * MI, ns = n0 + (wmn % WN) * 16 * NI;
    const bool out = ms >= p.M || ns >= p.N;
    const int mt = TA && MI > 1 ? min(ms, p.M - 16 * MI) : ms;
    const int nt = !TB && NI > 1 ? min(ns, p.N - 16 * NI) : ns;

    acc_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

    typedef Side<T, !TA, MI> SideA;
    typedef Side<T, TB, NI> SideB;
    if (!out) {
        SideA sa;
        SideB sb;
        T* mine = lds + wave * (SideA::LDS + SideB::LDS);
        sa.init(A, p.lda, mt, p.M, lane, mine);
        sb.init(B, p.ldb, nt, p.N, lane, mine + SideA::LDS);
        const int nk = (p.K + BK - 1) / BK;
        const int kb = KS == 1 ? 0 : (int)((long)nk * ks / KS), ke = KS == 1 ? nk : (int)((long)nk * (ks + 1) / KS);
        const int nfull = min(ke, p.K / BK) - kb;    // full slices of this part, from kb on
        typename SideA::Slice a[PD];
        typename SideB::Slice b[PD];
        T x[MI][4], y[NI][4];
        auto load = [&](int u, int kt) {
            sa.load((kb + kt) * BK, a[u]);
            sb.load((kb + kt) * BK, b[u]);
        };
        auto values = [&](int u) {
            sa.values(a[u], x);
            sb.values(b[u], y);
        };
        auto mma = [&] {
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j) acc[i][j] = MfmaOp<T>::mma(x[i][s], y[j][s], acc[i][j]);
        };
#pragma unroll
        for (int u = 0; u < PD; ++u)
            if (u < nfull) load(u, u);
        int kt = 0;
        for (; kt + 2 * PD <= nfull; kt += PD) {
#pragma unroll
            for (int u = 0; u < PD; ++u) {
                values(u);
                load(u, kt + PD + u);
                mma();
            }
        }
        // kt + PD <= nfull < kt + 2 PD, or nfull < PD
        const int left = nfull - kt;
#pragma unroll
        for (int u = 0; u < PD; ++u)
            if (u < left) {
                values(u);
                if (u + PD < left) load(u, kt + PD + u);
                mma();
            }
#pragma unroll
        for (int u = 0; u < PD; ++u)
            if (u + PD < left) {
                values(u);
                mma();
            }
        if (ke > kb && ke * BK > p.K) {
            sa.load_tail((ke - 1) * BK, p.K, a[0]);
            sb.load_tail((ke - 1) * BK, p.K, b[0]);
            values(0);
            mma();
        }
    }

    finish_tile<MI, NI, WM, WN, KS>(
        p, bz, ms, ns, out, acc, [&](int i, int r) { return mt + SideA::index(i, MfmaOp<T>::row(lane >> 4, r)); },
        [&](int j) { return nt + SideB::index(j, lane & 15); }, lds);
}

template <typename T, bool TA, bool TB, int MI, int NI, int WM, int WN, int KS, int PD>
__global__ __launch_bounds__(64 * WM * WN * KS) void direct_kernel(Params p) {
    __shared__ __attribute__((aligned(16))) T lds[direct_lds<T, TA, TB, MI, NI, WM, WN, KS>()];
    const int tile = xcd_band_tile(blockIdx.x, p.mt * p.nt);
    direct_tile<T, TA, TB, MI, NI, WM, WN, KS, PD>(p, (tile / p.nt) * 16 * MI * WM, (tile % p.nt) * 16 * NI * WN,
                                                   (long)blockIdx.z, lds);
}

// ---------------------------------------------------------------------------
// BF16 operands, FP32 accumulation: the same with slices of 64 (two
// v_mfma_f32_16x16x32_bf16 steps), lane group g supplying K values 8 g .. 8 g +
// 7 of a step.  Side-contiguous operands are packed from eight K rows in
// registers.
// ---------------------------------------------------------------------------
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
constexpr int BKB = 64;

template <bool KC, int S> struct SideB16;

template <int S> struct SideB16<true, S> {
    static constexpr int LDK = BKB + 8, LDS = 16 * S * LDK;   // in 16-bit words
    struct Slice { uint4 v[2 * S]; };
    const uint16_t* ptr[2 * S];
    uint16_t* lds;
    int lane;
    __device__ void init(const uint16_t* src, long ld, int side0, int sideN, int lane_, uint16_t* lds_) {
        lane = lane_;
        lds = lds_;
#pragma unroll
        for (int n = 0; n < 2 * S; ++n)
            ptr[n] = src + (long)min(side0 + 8 * n + (lane >> 3), sideN - 1) * ld + (lane & 7) * 8;
    }
    __device__ static int index(int t, int pos) { return 16 * t + pos; }
    __device__ static uint4 pack(const uint16_t (&h)[8]) {
        return uint4{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
                     (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16)};
    }
    __device__ void load(int k0, Slice& r) const {
#pragma unroll
        for (int n = 0; n < 2 * S; ++n) {
            uint16_t h[8];
            load_elems<uint16_t, 8>(ptr[n] + k0, h);
            r.v[n] = pack(h);
        }
    }
    __device__ void load_tail(int k0, int K, Slice& r) const {
#pragma unroll
        for (int n = 0; n < 2 * S; ++n) {
            uint16_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = k0 + (lane & 7) * 8 + e < K ? ptr[n][k0 + e] : (uint16_t)0;
            r.v[n] = pack(h);
        }
    }
    __device__ void values(const Slice& r, bf8_t (&v)[S][2]) const {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int n = 0; n < 2 * S; ++n)
            *reinterpret_cast<uint4*>(&lds[(8 * n + (lane >> 3)) * LDK + (lane & 7) * 8]) = r.v[n];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                v[i][h] = *reinterpret_cast<const bf8_t*>(&lds[(16 * i + (lane & 15)) * LDK + 32 * h + 8 * (lane >> 4)]);
    }
};

template <int S> struct SideB16<false, S> {
    static constexpr int LDS = 0;
    struct Slice { uint16_t v[16][S]; };
    const uint16_t* ptr;
    long ld;
    int kg;
    __device__ void init(const uint16_t* src, long ld_, int side0, int sideN, int lane, uint16_t*) {
        ld = ld_;
        kg = lane >> 4;
        const int l16 = lane & 15;
        ptr = src + (S == 1 ? min(side0 + l16, sideN - 1) : side0 + S * l16) + (long)(8 * kg) * ld;
    }
    __device__ static int index(int t, int pos) { return S * pos + t; }
    __device__ void load(int k0, Slice& r) const {
#pragma unroll
        for (int e = 0; e < 16; ++e) load_elems<uint16_t, S>(ptr + (long)(k0 + 32 * (e >> 3) + (e & 7)) * ld, r.v[e]);
    }
    __device__ void load_tail(int k0, int K, Slice& r) const {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int k = k0 + 32 * (e >> 3) + (e & 7);
#pragma unroll
            for (int i = 0; i < S; ++i) r.v[e][i] = k + 8 * kg < K ? ptr[(long)k * ld + i] : (uint16_t)0;
        }
    }
    __device__ void values(const Slice& r, bf8_t (&v)[S][2]) const {
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint4 x;
                uint32_t* w = &x.x;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] = (uint32_t)r.v[8 * h + 2 * e][i] | ((uint32_t)r.v[8 * h + 2 * e + 1][i] << 16);
                v[i][h] = *reinterpret_cast<const bf8_t*>(&x);
            }
    }
};

template <bool TA, bool TB, int MI, int NI, int WM, int WN, int KS>
__global__ __launch_bounds__(64 * WM * WN * KS) void direct_bf16_kernel(Params p) {
    typedef SideB16<!TA, MI> SideA;
    typedef SideB16<TB, NI> SideB;
    constexpr int STAGE = WM * WN * KS * (SideA::LDS + SideB::LDS) / 2, PARTS = KS == 1 ? 1 : KS * WM * WN * MI * NI * 256;
    __shared__ __attribute__((aligned(16))) float lds[STAGE > PARTS ? STAGE : PARTS];
    const int tile = xcd_band_tile(blockIdx.x, p.mt * p.nt);
    const long bz = blockIdx.z;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = wave / (WM * WN), wmn = wave % (WM * WN);
    const int ms = ((tile / p.nt) * WM + wmn / WN) * 16 * MI, ns = ((tile % p.nt) * WN + wmn % WN) * 16 * NI;
    const bool out = ms >= p.M || ns >= p.N;
    const int mt = TA && MI > 1 ? min(ms, p.M - 16 * MI) : ms;
    const int nt = !TB && NI > 1 ? min(ns, p.N - 16 * NI) : ns;
    f4_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = f4_t{0, 0, 0, 0};
    if (!out) {
        SideA sa;
        SideB sb;
        uint16_t* mine = reinterpret_cast<uint16_t*>(lds) + wave * (SideA::LDS + SideB::LDS);
        sa.init(static_cast<const uint16_t*>(p.A) + bz * p.sA, p.lda, mt, p.M, lane, mine);
        sb.init(static_cast<const uint16_t*>(p.B) + bz * p.sB, p.ldb, nt, p.N, lane, mine + SideA::LDS);
        const int nk = (p.K + BKB - 1) / BKB;
        const int kb = (int)((long)nk * ks / KS), ke = (int)((long)nk * (ks + 1) / KS);
        typename SideA::Slice a;
        typename SideB::Slice b;
        auto load = [&](int kt) {
            if ((kt + 1) * BKB <= p.K) {
                sa.load(kt * BKB, a);
                sb.load(kt * BKB, b);
            } else {
                sa.load_tail(kt * BKB, p.K, a);
                sb.load_tail(kt * BKB, p.K, b);
            }
        };
        if (kb < ke) load(kb);
        for (int kt = kb; kt < ke; ++kt) {
            bf8_t x[MI][2], y[NI][2];
            sa.values(a, x);
            sb.values(b, y);
            if (kt + 1 < ke) load(kt + 1);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i][h], y[j][h], acc[i][j], 0, 0, 0);
        }
    }
    finish_tile<MI, NI, WM, WN, KS>(
        p, bz, ms, ns, out, acc, [&](int i, int r) { return mt + SideA::index(i, 4 * (lane >> 4) + r); },
        [&](int j) { return nt + SideB::index(j, lane & 15); }, lds);
}

}  // namespace
}  // namespace ite
