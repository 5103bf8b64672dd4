// MFMA GEMM for gfx950 (CDNA4): the contraction core of the
// effective-Hamiltonian product and of the environment updates.
//
// D[b] = alpha op(A[b]) op(B[b]) + beta C[b], row-major.
//
// FP64 and FP32 operands: gemm_direct.h (memory -> registers -> matrix cores,
// no barrier in the K loop), with the wavefront and workgroup tiles chosen by
// tile_kind.  BF16 operands: the same, or a 128 x 128 tile staged through LDS.
//
// Workgroup -> tile mapping is XCD-aware: the hardware deals workgroups to the
// 8 XCDs round-robin, so consecutive workgroup ids are remapped to give each
// XCD a contiguous band of output tiles that share A row panels in that XCD's
// L2.
#include "gemm_direct.h"
#include "gemm_tile.h"
#include "internal.h"

#include <algorithm>
#include <climits>
#include <cstdint>
#include <cstring>
#include <type_traits>

namespace ite {
namespace {

template <typename T, int MI, int NI, int WM, int WN, int KS, int PD>
void launch_tiles(const Gemm& g, Params p, hipStream_t s) {
    p.mt = (g.M + 16 * MI * WM - 1) / (16 * MI * WM);
    p.nt = (g.N + 16 * NI * WN - 1) / (16 * NI * WN);
    const dim3 grid(p.mt * p.nt, 1, g.batch), block(64 * WM * WN * KS);
#define ITE_GL(TA, TB) hipLaunchKernelGGL((direct_kernel<T, TA, TB, MI, NI, WM, WN, KS, PD>), grid, block, 0, s, p)
    if (!g.tA && !g.tB) ITE_GL(false, false);
    else if (!g.tA && g.tB) ITE_GL(false, true);
    else if (g.tA && !g.tB) ITE_GL(true, false);
    else ITE_GL(true, true);
#undef ITE_GL
    HIP_CHECK(hipGetLastError());
}

// Tile of a product, by its shape alone (a problem of a grouped launch has the
// bits it has alone).  A matrix-core step takes a wavefront 64 cycles (FP64)
// or 32 (FP32), so one accumulator chain keeps a SIMD's matrix core busy; what
// matters is that every SIMD has a wavefront and that operands are read few
// times.  Larger tiles read less (a 64 x 64 workgroup 1/4 of a 16 x 16 one),
// smaller tiles and K parts fill the chip when the output is small.
//
// FP64 (us; 16: 16 x 16 with 4 or 8 K parts, 32: 32 x 32 with 8, 64: 64 x 64
// with 2; LDS: 128 x 128 tiles staged through LDS with a barrier a slice,
// which all of these replace):
//      M x N x K                16      32      64     LDS
//      128 x 32 x 160  (NT)    3.4     5.3     9.9    31.5
//      480 x 120 x 600 (NT)    5.5    10.0    28.4     105
//      400 x 400 x 200         5.9     6.2    12.4    45.7     169 32-tiles
//      512 x 512 x 256         6.7     6.1    13.5    52.8     256 32-tiles
//      1024 x 256 x 1280 (NT) 19.3    17.7    56.5     211     256 32-tiles
//      1280 x 1024 x 256        33    20.1    24.2      66     320 64-tiles
//      1920 x 1536 x 384        74    56.5    47.7      87     720 64-tiles
//      5120 x 4096 x 1024     1550     895     694     829
// so 64 from 512 of its tiles on (two workgroups a compute unit), 32 from 192
// of its tiles on.  A few tiles more than 512 are a second round that leaves most
// of the chip idle, which costs more the longer K is (H_eff, us, its second product in
// 32 and 64: 576 tiles, K 3840 730 and 858; 676, K 4160 927 and 993; 756, K 4320 1029 and
// 1068; 784, K 4480 1148 and 1156; 900, K 4800 1412 and 1367): with a long K 64 at
// 512, where the one round is full, and from 800 on (NN, us with the call: 496 tiles, K
// 2048 170 and 149; 512 212 and 149, K 1024 100 and 84; 528, K 2048 188 and 211).  With 16, four K parts are as fast as eight while K is
// short (160 x 128 x 32: 2.9 and 3.4) and slower when it is long (64 x 64 x
// 4000: 18.1 and 13.4); they meet near 500.
//
// FP32 (us; the 32 tile with 4 K parts):
//      480 x 120 x 600 (NT)    4.6     7.7    16.5    67.2
//      600 x 480 x 120         5.6     5.5     7.9    26.3     285 32-tiles
//      1024 x 256 x 1280 (NT) 12.8    12.1    29.1     126     256 32-tiles
//      1532 x 401 x 2005 (NT) 53.7    39.1    46.3     201     168 64-tiles
//      1920 x 1536 x 384      49.4    31.0    31.7    61.4     720 64-tiles
//      2560 x 2048 x 512       110    66.9    62.7     106    1280 64-tiles
//      5120 x 4096 x 1024      938     562     458     561
// the same, with 64 from 1024 of its tiles on.
//
// Up to a K of 128 the exchange of the two K parts costs a 64 tile more than they
// save: it has one part there (us with the call and its wait, some 20: two parts,
// one, and LDS as above; NN):
//      4336 x 1880 x 16       34  30  29    FP32  34  33  33
//      2500 x 7500 x 32       69  62  61          56  53  53
//      4000 x 4000 x 100     108  94  95          76  72  86
//      6850 x 2468 x 128     114 105 124          79  74  97
//      2048 x 2048 x 256      56  57  61          48  46  53
//      4000 x 4000 x 512     307 324 316         204 187 234
// (FP32 keeps two parts beyond 128 as well, for the shorter chains of additions.)
//
// A side-contiguous operand (A transposed, B not) needs a side of at least
// one wavefront tile, which only the 16-wide tiles guarantee.
template <typename T> constexpr int K32 = sizeof(T) == 8 ? 8 : 4;   // K parts of the 32 tile
constexpr int K_SHORT = 128;
enum TileKind { TILE_64, TILE_64_SHORT, TILE_32, TILE_16_LONG, TILE_16 };
template <typename T>
TileKind tile_kind(const Gemm& g) {
    auto tiles = [&](int side) { return (long)((g.M + side - 1) / side) * ((g.N + side - 1) / side) * g.batch; };
    const bool wide = (!g.tA || g.M >= 32) && (g.tB || g.N >= 32);
    const long t64 = tiles(64);
    if (wide && t64 >= (!std::is_same<T, double>::value ? 1024 : g.K >= 1024 && t64 > 512 ? 800 : 512))
        return g.K <= K_SHORT ? TILE_64_SHORT : TILE_64;
    if (wide && tiles(32) >= 192) return TILE_32;
    return g.K >= 512 ? TILE_16_LONG : TILE_16;
}

// Large TILE_64 products take larger tiles of the same two K parts (the same
// bits, so a grouped launch need not): wavefronts of 32 x 64 (FP64) or 64 x 64
// (FP32) read 3/4 or half of what those of 32 x 32 do, and one workgroup fills
// a compute unit.
//
// H_eff products, us of both of their products and the stage (none / 2048 tiles on / 1024 on):
//      d 2, bond 512, FP64 (1280 tiles, K 512)              224     224     241
//      d 4, bond 384, FP64 (3456 tiles, K 384)              553     570     568
//      d 2, bond 1024, FP64 (5120, K 1024; 1024, K 5120)   1608    1577    1508
//      d 2, bond 512, FP32                                  127     128     132
//      d 2, bond 768, FP32 (2880 tiles, K 768)              412     385     385
//      d 4, bond 512, FP32 (6144, K 512; 1024, K 3072)      584     542     526
// so a long K pays from 1024 tiles on in either type, one of 512 or more in FP32
// from 2048 on (below 512 the 64 x 64 tile is faster, FP32, NN, us with the call:
// 2500 x 7500 x 32 82 and 56, x 128 115 and 91, x 256 156 and 140, x 384 195 and 190,
// x 512 230 and 239).  Around the FP64 line a whole product takes, without and with
// them (d 2, us, forty in a row): bond 896 1127 and 1147, 960 1302 and 1308, 1000 1521
// and 1453 (not taken: 1008 tiles), 1024 1533 and 1483, 1056 1862 and 1917, 1088 1980
// and 2036, 1152 2252 and 2239, 1280 3078 and 3183, 1400 4155 and 3792, 1536 5256 and
// 5044: where the last round of tiles is nearly full they win by up to 9%, where it is
// nearly empty they lose 3%.  Not in FP64 with A transposed (environment updates up to bond 1024,
// on average 391 and 457 us).
template <typename T>
bool large_tile(const Gemm& g) {
    const long tiles = (long)((g.M + 63) / 64) * ((g.N + 63) / 64) * g.batch;
    if ((g.tA && (std::is_same<T, double>::value || g.M < 64)) || (!g.tB && g.N < 64)) return false;
    return tiles >= (g.K >= 1024 ? 1024 : std::is_same<T, double>::value || g.K < 512 ? LONG_MAX : 2048);
}

Params params(const Gemm& g) {
    Params p{};
    p.M = g.M; p.N = g.N; p.K = std::max(g.K, 0);
    p.alpha = g.alpha; p.beta = g.beta;
    p.A = g.A; p.lda = g.lda; p.sA = g.sA;
    p.B = g.B; p.ldb = g.ldb; p.sB = g.sB;
    p.C = g.C; p.ldc = g.ldc; p.sC = g.sC;
    p.D = g.D; p.ldd = g.ldd; p.sD = g.sD;
    p.Df = g.Df;
    return p;
}

template <typename T>
void launch(const Gemm& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return;
    if (g.Df && g.C) ITE_FAIL(ITE_EINVAL, "gemm: an FP32 output takes no C");
    Params p = params(g);
    if (std::is_same<T, double>::value) p.Df = nullptr;
    const TileKind kind = tile_kind<T>(g);
    if (kind == TILE_64 && large_tile<T>(g)) {
        if constexpr (std::is_same<T, double>::value) launch_tiles<T, 2, 4, 2, 2, 2, 1>(g, p, s);
        else launch_tiles<T, 4, 4, 2, 1, 2, 1>(g, p, s);
    } else if (kind == TILE_64) launch_tiles<T, 2, 2, 2, 2, 2, 1>(g, p, s);
    else if (kind == TILE_64_SHORT) launch_tiles<T, 2, 2, 2, 2, 1, 1>(g, p, s);
    else if (kind == TILE_32) launch_tiles<T, 2, 2, 1, 1, K32<T>, 1>(g, p, s);
    else if (kind == TILE_16_LONG) launch_tiles<T, 1, 1, 1, 1, 8, 2>(g, p, s);
    else launch_tiles<T, 1, 1, 1, 1, 4, 2>(g, p, s);
}

// Many independent problems in one persistent launch (the products of the
// requests batched by the serving path): problem g's tiles are
// [tile_start[g], tile_start[g + 1]) of a common range, row-major over its
// output; every workgroup walks that range with a stride of the grid, so the
// grid can stay fixed (graph capture) while the problems change.  The
// descriptors live in device memory.  Each problem has the tile of its shape;
// one of four wavefronts takes two neighbours for the eight.
struct GroupDesc {
    Params p;
    int tile_start;
    int kind;
};
int group_rows(TileKind k) { return k == TILE_64 || k == TILE_64_SHORT ? 64 : k == TILE_32 ? 32 : 16; }
int group_cols(TileKind k, bool f32) {
    return k == TILE_64 ? 64 : k == TILE_64_SHORT ? 128 : k == TILE_32 ? (f32 ? 64 : 32) : k == TILE_16_LONG ? 16 : 32;
}

template <typename T, bool TB>
__global__ __launch_bounds__(512) void gemm_grouped_kernel(const GroupDesc* __restrict__ desc,
                                                           const int* __restrict__ count) {
    constexpr int W32 = 8 / K32<T>;
    constexpr int L64 = direct_lds<T, false, TB, 2, 2, 2, 2, 2>(), L32 = direct_lds<T, false, TB, 2, 2, 1, W32, K32<T>>();
    __shared__ __attribute__((aligned(16))) T lds[L64 > L32 ? L64 : L32];
    const int G = count[0], ntiles = count[1];
    int g = 0;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        while (g + 1 < G && desc[g + 1].tile_start <= tile) ++g;
        const Params p = desc[g].p;
        const int kind = desc[g].kind;
        const int lt = tile - desc[g].tile_start, m = lt / p.nt, n = lt % p.nt;
        if (kind == TILE_64) direct_tile<T, false, TB, 2, 2, 2, 2, 2, 1>(p, m * 64, n * 64, 0, lds);
        else if (kind == TILE_64_SHORT) direct_tile<T, false, TB, 2, 2, 2, 4, 1, 1>(p, m * 64, n * 128, 0, lds);
        else if (kind == TILE_32) direct_tile<T, false, TB, 2, 2, 1, W32, K32<T>, 1>(p, m * 32, n * 32 * W32, 0, lds);
        else if (kind == TILE_16_LONG) direct_tile<T, false, TB, 1, 1, 1, 1, 8, 2>(p, m * 16, n * 16, 0, lds);
        else direct_tile<T, false, TB, 1, 1, 1, 2, 4, 2>(p, m * 16, n * 32, 0, lds);
        __syncthreads();   // the LDS is the next tile's
    }
}

// One v_mfma_f64_16x16x4f64 with A[i][k] = 1 + i + 16 k (i < 16, k < 4)
// supplied by lane i + 16 k and B[k][j] = 1 / (1 + j + 16 k) by lane j + 16 k;
// every lane writes its four accumulator values.
__global__ void mfma_probe_kernel(double* out) {
    const int l = threadIdx.x;
    const double a = 1.0 + (l & 15) + 16.0 * (l >> 4);
    const double b = 1.0 / (1.0 + (l & 15) + 16.0 * (l >> 4));
    d4_t acc = {0, 0, 0, 0};
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
    for (int r = 0; r < 4; ++r) out[l * 4 + r] = acc[r];
}

// ---------------------------------------------------------------------------
// BF16 operands, FP32 accumulation: v_mfma_f32_16x16x32_bf16 (gfx950).  Same
// 128 x 128 tile and 2 x 2 wave arrangement as above; K advances in slices of
// 64 (two MFMA K steps per 16 x 16 tile, 32 MFMAs per wave between barriers).
// Both operands sit in LDS as [row][64 K values] (row = output row or
// column), in 16-byte chunks of 8 K values whose position within the row is
// XOR-swizzled by the row index, so that the MFMA reads (16 rows, one chunk
// each) and the transposing writes of a side-contiguous operand spread over
// the banks without padding.  Lane group g = lane / 16 supplies K values
// 8 g .. 8 g + 7 of each 32-wide step; A and B use the same mapping.
// ---------------------------------------------------------------------------
constexpr int BK16 = 64;

// u16 offset of chunk c (8 K values) of LDS row r
__device__ inline int swz16(int r, int c) { return r * BK16 + ((c ^ (r & 7) ^ ((r >> 3) & 7)) << 3); }

// Registers of one operand's K slice: four 16-byte words per thread.
struct Slice16 {
    uint4 v[4];
};

// K-contiguous source ([side][K]): thread t fetches chunks u = t + 256 e,
// row u / 8, chunk u % 8 (eight threads read one row's 128 bytes).
template <bool VEC>
__device__ inline void fetch16_kc(const uint16_t* __restrict__ src, long ld, int side0, int sideN, int k0, int K,
                                  int t, Slice16& r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int u = t + 256 * e;
        const int row = side0 + (u >> 3);
        const int k = k0 + (u & 7) * 8;
        if (VEC && row < sideN && k + 7 < K) {
            r.v[e] = *reinterpret_cast<const uint4*>(src + (long)row * ld + k);
        } else {
            uint16_t h[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) h[q] = (row < sideN && k + q < K) ? src[(long)row * ld + k + q] : (uint16_t)0;
            r.v[e] = uint4{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
                           (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16)};
        }
    }
}
__device__ inline void store16_kc(uint16_t* __restrict__ lds, int t, const Slice16& r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int u = t + 256 * e;
        *reinterpret_cast<uint4*>(&lds[swz16(u >> 3, u & 7)]) = r.v[e];
    }
}

// Side-contiguous source ([K][side]): thread t fetches a 4 (K) x 8 (side)
// block, K rows 4 (t / 16) .. +3 and side values 8 (t % 16) .. +7 (sixteen
// threads read one K row's 256 bytes), and writes it transposed: eight LDS
// rows of four K values (8 bytes each).
template <bool VEC>
__device__ inline void fetch16_sc(const uint16_t* __restrict__ src, long ld, int side0, int sideN, int k0, int K,
                                  int t, Slice16& r) {
    const int col = side0 + (t & 15) * 8;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = k0 + (t >> 4) * 4 + e;
        if (VEC && k < K && col + 7 < sideN) {
            r.v[e] = *reinterpret_cast<const uint4*>(src + (long)k * ld + col);
        } else {
            uint16_t h[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) h[q] = (k < K && col + q < sideN) ? src[(long)k * ld + col + q] : (uint16_t)0;
            r.v[e] = uint4{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
                           (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16)};
        }
    }
}
__device__ inline uint32_t word16(const uint4& v, int q) {
    const uint32_t w = q < 2 ? (q == 0 ? v.x : v.y) : (q == 2 ? v.z : v.w);
    return w;
}
__device__ inline void store16_sc(uint16_t* __restrict__ lds, int t, const Slice16& r) {
    const int s0 = (t & 15) * 8;
    const int kb = t >> 4;   // K values 4 kb .. 4 kb + 3: chunk kb / 2, half kb % 2
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t a0 = word16(r.v[0], w), a1 = word16(r.v[1], w);
        const uint32_t a2 = word16(r.v[2], w), a3 = word16(r.v[3], w);
        // side value 2 w (low halves) and 2 w + 1 (high halves)
        const uint2 lo{(a0 & 0xffffu) | (a1 << 16), (a2 & 0xffffu) | (a3 << 16)};
        const uint2 hi{(a0 >> 16) | (a1 & 0xffff0000u), (a2 >> 16) | (a3 & 0xffff0000u)};
        *reinterpret_cast<uint2*>(&lds[swz16(s0 + 2 * w, kb >> 1) + (kb & 1) * 4]) = lo;
        *reinterpret_cast<uint2*>(&lds[swz16(s0 + 2 * w + 1, kb >> 1) + (kb & 1) * 4]) = hi;
    }
}

template <bool KC, bool VEC>
__device__ inline void fetch16(const uint16_t* __restrict__ src, long ld, int side0, int sideN, int k0, int K, int t,
                               Slice16& r) {
    if constexpr (KC) fetch16_kc<VEC>(src, ld, side0, sideN, k0, K, t, r);
    else fetch16_sc<VEC>(src, ld, side0, sideN, k0, K, t, r);
}
template <bool KC>
__device__ inline void store16(uint16_t* __restrict__ lds, int t, const Slice16& r) {
    if constexpr (KC) store16_kc(lds, t, r);
    else store16_sc(lds, t, r);
}

template <bool TA, bool TB, bool VEC>
__global__ __launch_bounds__(NTHREADS) void gemm_bf16_kernel(Params p) {
    __shared__ __attribute__((aligned(16))) uint16_t As[2][BM * BK16];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[2][BN * BK16];
    const int T_tiles = p.mt * p.nt;
    const int tile = xcd_band_tile(blockIdx.x, T_tiles);
    const int m0 = (tile / p.nt) * BM;
    const int n0 = (tile % p.nt) * BN;
    const long bz = blockIdx.z;
    const uint16_t* __restrict__ A = static_cast<const uint16_t*>(p.A) + bz * p.sA;
    const uint16_t* __restrict__ B = static_cast<const uint16_t*>(p.B) + bz * p.sB;
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l16 = lane & 15, kg = lane >> 4;
    f4_t acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f4_t{0, 0, 0, 0};
    Slice16 ra, rb;
    const int nk = (p.K + BK16 - 1) / BK16;
    fetch16<!TA, VEC>(A, p.lda, m0, p.M, 0, p.K, t, ra);
    fetch16<TB, VEC>(B, p.ldb, n0, p.N, 0, p.K, t, rb);
    store16<!TA>(As[0], t, ra);
    store16<TB>(Bs[0], t, rb);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        const bool more = kt + 1 < nk;
        if (more) {
            fetch16<!TA, VEC>(A, p.lda, m0, p.M, (kt + 1) * BK16, p.K, t, ra);
            fetch16<TB, VEC>(B, p.ldb, n0, p.N, (kt + 1) * BK16, p.K, t, rb);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf8_t a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                a[i] = *reinterpret_cast<const bf8_t*>(&As[cur][swz16(wm * 64 + i * 16 + l16, 4 * h + kg)]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                b[j] = *reinterpret_cast<const bf8_t*>(&Bs[cur][swz16(wn * 64 + j * 16 + l16, 4 * h + kg)]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (more) {
            store16<!TA>(As[cur ^ 1], t, ra);
            store16<TB>(Bs[cur ^ 1], t, rb);
        }
        __syncthreads();
    }
    const double* __restrict__ C = p.C ? p.C + bz * p.sC : nullptr;
    double* __restrict__ D = p.Df ? nullptr : p.D + bz * p.sD;
    float* __restrict__ Df = p.Df ? p.Df + bz * p.sD : nullptr;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = n0 + wn * 64 + j * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm * 64 + i * 16 + 4 * kg + r;
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

void gemm_f64(const Gemm& g, hipStream_t s) { launch<double>(g, s); }

namespace {
// Operands fit 16-byte loads: aligned bases, row strides and batch strides
// that are multiples of 16 bytes.
inline bool vec16(const Gemm& g, size_t esz) {
    const size_t q = 16 / esz;
    auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
    return al(g.A) && al(g.B) && g.lda % q == 0 && g.ldb % q == 0 && g.sA % q == 0 && g.sB % q == 0;
}

// D[m][n] = alpha sum_b W[b][m][n] + beta C[m][n], the parts summed in order.
__global__ __launch_bounds__(256) void splitk_sum_kernel(const double* __restrict__ W, int parts, int M, int N,
                                                         double alpha, const double* C, long ldc, double beta,
                                                         double* D, long ldd) {
    const long n_all = (long)M * N, part = n_all;
    for (long e = blockIdx.x * 256L + threadIdx.x; e < n_all; e += (long)gridDim.x * 256) {
        double v = W[e];
        for (int b = 1; b < parts; ++b) v += W[b * part + e];
        const long m = e / N, n = e % N;
        v *= alpha;
        if (C) v += beta * C[m * ldc + n];
        D[m * ldd + n] = v;
    }
}
}  // namespace

// Eight K parts of a workgroup are enough until each is 32 slices of 16 long;
// beyond that more workgroups share K.
int splitk_parts(int M, int N, int K) {
    const long tiles = (long)((M + 15) / 16) * ((N + 15) / 16);
    if (tiles > 128 || K < 4096) return 1;
    int s = (int)std::min<long>(256 / tiles, K / 2048);
    while (s > 1 && K % (s * BK) != 0) --s;
    return std::max(s, 1);
}

// The K parts of g (no C, alpha 1) as one batched launch: part k to
// out + k part_stride (FP64) with row stride ldo.
template <typename T>
static void gemm_kparts(const Gemm& g, int parts, double* out, long ldo, long part_stride, hipStream_t s) {
    if (g.batch != 1 || g.Df) ITE_FAIL(ITE_EINVAL, "gemm K parts: single problems with an FP64 output only");
    if (parts < 1 || g.K % parts != 0) ITE_FAIL(ITE_EINVAL, "gemm K parts: K must split evenly");
    const int kp = g.K / parts;
    Gemm h = g;
    h.K = kp;
    h.batch = parts;
    h.sA = g.tA ? (long)kp * g.lda : kp;      // A stored K x M when transposed, else M x K
    h.sB = g.tB ? kp : (long)kp * g.ldb;      // B stored N x K when transposed, else K x N
    h.alpha = 1.0;
    h.beta = 0.0;
    h.C = nullptr;
    h.D = out;
    h.ldd = ldo;
    h.sD = part_stride;
    launch<T>(h, s);
}

template <typename T>
static void gemm_splitk(const Gemm& g, int parts, double* work, hipStream_t s) {
    if (parts <= 1) {
        launch<T>(g, s);
        return;
    }
    gemm_kparts<T>(g, parts, work, g.N, (long)g.M * g.N, s);
    const long n = (long)g.M * g.N;
    const int grid = (int)std::min<long>(4096, (n + 255) / 256);
    hipLaunchKernelGGL(splitk_sum_kernel, dim3(grid), dim3(256), 0, s, work, parts, g.M, g.N, g.alpha, g.C, g.ldc,
                       g.beta, g.D, g.ldd);
    HIP_CHECK(hipGetLastError());
}

void gemm_f64_splitk(const Gemm& g, int parts, double* work, hipStream_t s) { gemm_splitk<double>(g, parts, work, s); }
void gemm_f32_splitk(const Gemm& g, int parts, double* work, hipStream_t s) { gemm_splitk<float>(g, parts, work, s); }

size_t grouped_desc_bytes() { return sizeof(GroupDesc); }

// Host side of a grouped launch: the descriptor of problem g (its tiles
// start at tile_start) in the layout gemm_grouped_kernel reads; returns the
// number of its tiles.
int grouped_desc_fill(const Gemm& g, bool f32, int tile_start, void* out) {
    const TileKind k = f32 ? tile_kind<float>(g) : tile_kind<double>(g);
    GroupDesc d{};
    d.p = params(g);
    d.p.sA = d.p.sB = d.p.sC = d.p.sD = 0;
    d.p.mt = g.M > 0 ? (g.M + group_rows(k) - 1) / group_rows(k) : 0;
    d.p.nt = g.N > 0 ? (g.N + group_cols(k, f32) - 1) / group_cols(k, f32) : 0;
    d.tile_start = tile_start;
    d.kind = k;
    std::memcpy(out, &d, sizeof(d));
    return d.p.mt * d.p.nt;
}

void gemm_grouped(const void* desc, const int* count, bool f32, bool tB, hipStream_t s) {
    const auto* d = static_cast<const GroupDesc*>(desc);
    const dim3 grid(512);
    if (f32) {
        if (tB) hipLaunchKernelGGL((gemm_grouped_kernel<float, true>), grid, dim3(512), 0, s, d, count);
        else hipLaunchKernelGGL((gemm_grouped_kernel<float, false>), grid, dim3(512), 0, s, d, count);
    } else {
        if (tB) hipLaunchKernelGGL((gemm_grouped_kernel<double, true>), grid, dim3(512), 0, s, d, count);
        else hipLaunchKernelGGL((gemm_grouped_kernel<double, false>), grid, dim3(512), 0, s, d, count);
    }
    HIP_CHECK(hipGetLastError());
}

void gemm_f32(const Gemm& g, hipStream_t s) { launch<float>(g, s); }

// BF16 tiles: straight to registers (32 x 32 or 16 x 16, four K parts) while the
// 128 x 128 tiles through LDS leave compute units idle; those read each operand
// a quarter as often and win once they fill the chip, from 256 of them on:
// 16 x 16, 32 x 32 and LDS 128, us on the device
//      128 x 32 x 160 (NT)       4.1   6.5  13.7
//      2048 x 128 x 768 (NT)     4.9   5.2  24.2     256 32-tiles
//      4096 x 256 x 1536 (NT)   19.6  14.3  38.5      64 128-tiles
// and the latter two with the call and its wait, some 20 us (NN, NT, TN):
//      1024 x 1024 x 512         27 33   27 33   28 34      64
//      2048 x 1024 x 512         34 37   33 37   36 38     128
//      1920 x 1536 x 512         38 37   36 36   40 37     180
//      1920 x 1536 x 2048        82 65   71 63   93 66     180
//      2048 x 2048 x 256         35 32   35 31   36 32     256
//      2048 x 2048 x 2048       115 68  104 66  126 69     256
//      6361 x 704 x 1024         62 67   57 62      --     300
//      1536 x 4096 x 256         43 36   43 36   46 37     384
//      3000 x 2400 x 512         55 49   54 46   66 52     456
// From 160 on they win when K is long, and from 128 on when it is shorter than a
// slice of the 32 x 32 tile (2048 x 1024 x 32: 32 29  39 29  28 28).  Their loads
// are single values where an operand does not allow 16 bytes at a time, which
// takes longer the longer K is: such products go to LDS from 512 of these tiles
// on only, or 256 with K contiguous in both operands (2300 x 1840 x 512, TN, rows
// of 2300: 53 and 91; x 32: 36 and 31).
void gemm_bf16(const Gemm& g, hipStream_t s) {
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return;
    if (g.Df && g.C) ITE_FAIL(ITE_EINVAL, "gemm: an FP32 output takes no C");
    Params p = params(g);
    auto tiles = [&](int side) { return (long)((g.M + side - 1) / side) * ((g.N + side - 1) / side) * g.batch; };
    const bool wide = (!g.tA || g.M >= 32) && (g.tB || g.N >= 32);
    const bool v = vec16(g, sizeof(uint16_t));
    const long t128 = tiles(128);
    const bool lds = t128 >= (v || (!g.tA && g.tB) ? 256 : 512) || (t128 >= 160 && v && g.K >= 2048) ||
                     (t128 >= 128 && g.K < BKB);
    const int side = lds ? 128 : wide && tiles(32) >= 192 ? 32 : 16;
    p.mt = (g.M + side - 1) / side;
    p.nt = (g.N + side - 1) / side;
    const dim3 grid(p.mt * p.nt, 1, g.batch);
#define ITE_GB(TA, TB)                                                                                          \
    if (side == 16) hipLaunchKernelGGL((direct_bf16_kernel<TA, TB, 1, 1, 1, 1, 4>), grid, dim3(256), 0, s, p);  \
    else if (side == 32)                                                                                        \
        hipLaunchKernelGGL((direct_bf16_kernel<TA, TB, 2, 2, 1, 1, 4>), grid, dim3(256), 0, s, p);              \
    else if (v) hipLaunchKernelGGL((gemm_bf16_kernel<TA, TB, true>), grid, dim3(NTHREADS), 0, s, p);            \
    else hipLaunchKernelGGL((gemm_bf16_kernel<TA, TB, false>), grid, dim3(NTHREADS), 0, s, p)
    if (!g.tA && !g.tB) { ITE_GB(false, false); }
    else if (!g.tA && g.tB) { ITE_GB(false, true); }
    else if (g.tA && !g.tB) { ITE_GB(true, false); }
    else { ITE_GB(true, true); }
#undef ITE_GB
    HIP_CHECK(hipGetLastError());
}

void mfma_probe_f64(double* out, hipStream_t s) {
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(1), dim3(64), 0, s, out);
    HIP_CHECK(hipGetLastError());
}

}  // namespace ite
