// H_eff of a small block in one launch.
//
//   X1[(a' w), (s t c)] = L[(a' w), a] theta[a, (s t c)]
//   X3[a'][(p q u)][c]  = WW[(p q u), (w s t)] X1[a'][(w s t)][c]
//   y[(a' p q), c']     = beta X3[(a' p q), (u c)] R[c', (u c)]^T + alpha C
//
// As three launches a small block is bound by their latency: 3 us each for less
// than a microsecond of work in all, and a local solve is a chain of eleven such
// products.  Here a workgroup takes g rows a' through all three stages, with X1
// and X3 in LDS; g is as large as one 16-row matrix-core tile allows in both
// products.  What is asked of memory comes first, so that one latency covers
// theta, L, R and the matrix; then the matrix-core steps of two wavefronts a SIMD
// and the stage's LDS reads bound it (us a product in a row of them, one launch
// and three: d 2, w 5, bond 16 6.1 and 8.8, 32 8.1 and 9.6, 48 11.8 and 9.8; d 4,
// w 6, bond 16 8.6 and 10.5, 24 12.8 and 11.3).
#include "internal.h"
#include "units.h"

#include <algorithm>
#include <cstring>

namespace ite {
namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef double d2u_t __attribute__((ext_vector_type(2), aligned(8)));

constexpr int NW = 8, NT = 64 * NW;
constexpr size_t LDS_MAX = 96 * 1024;

// LDS of a workgroup, in doubles: L's rows, X1 (later the K parts of y), X3, the
// CSR matrix.
struct Shape {
    int I, O, N1, K3, ldl, ldx3, parts;
    int x1, x3, csr, total;
};
Shape shape_of(int Dyl, int Dxr, int Dyr, int w0, int w2, int dd, int g, int nnz) {
    Shape s;
    s.I = w0 * dd;
    s.O = dd * w2;
    s.N1 = dd * Dyr;
    s.K3 = w2 * Dyr;
    // even, so that the 16-byte reads of a row are aligned, and not a multiple of 16
    s.ldl = (Dyl + 15) / 16 * 16 + 2;
    s.ldx3 = (s.K3 + 15) / 16 * 16 + 2;
    const int t3 = (Dxr + 15) / 16;
    s.parts = t3 >= NW ? 1 : NW / t3;          // K parts of y
    s.x1 = 16 * s.ldl;
    s.x3 = s.x1 + (g * w0 * s.N1 > NW * 256 ? g * w0 * s.N1 : NW * 256);
    s.csr = s.x3 + 16 * s.ldx3;
    s.total = s.csr + nnz + (nnz + 2 * s.O + 3) / 2;
    return s;
}

struct Desc {
    const double *L, *theta, *R, *C;
    double* y;
    double alpha, beta;
    int Dxl, Dyl, Dxr, Dyr, w0, w2, dd, g;
    const int *rowptr, *col;
    const double* val;
    int nnz, start;
    Shape s;
};

__device__ inline void heff_tile(const Desc& h, int blk, double* lds) {
    const Shape& s = h.s;
    const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int a0 = blk * h.g, ga = min(h.g, h.Dxl - a0);
    double *Ls = lds, *x1 = lds + s.x1, *x3 = lds + s.x3;
    double* sval = lds + s.csr;
    int* scol = reinterpret_cast<int*>(sval + h.nnz);
    int* srow = scol + h.nnz;
    int* soff = srow + s.O + 1;                // where output o starts in a row of X3

    const int m1 = ga * h.w0, k1 = (h.Dyl + 15) / 16 * 16, k3 = (s.K3 + 15) / 16 * 16;
    // everything that comes from memory is asked for first.  theta: a column tile
    // a wavefront at a time, two slices in flight
    const int t1 = (s.N1 + 15) / 16, n1 = k1 / 16;
    int ftile = wave, fslice = 0;              // the next slice to fetch
    double b[2][4];
    auto fetch = [&](double (&v)[4]) {
        const int n = min(ftile * 16 + l16, s.N1 - 1), k0 = fslice * 16 + 4 * kg;
        const double* from = h.theta + (long)k0 * s.N1 + n;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = k0 + q < h.Dyl ? from[(long)q * s.N1] : 0.0;
        if (++fslice == n1) {
            fslice = 0;
            ftile += NW;
        }
    };
    if (ftile < t1) fetch(b[0]);
    if (ftile < t1) fetch(b[1]);
    // the first slices of R for this wavefront's part of y
    const int t3 = (h.Dxr + 15) / 16, n3 = k3 / 16;
    const int part = s.parts > 1 ? wave % s.parts : 0, tile0 = s.parts > 1 ? wave / s.parts : wave;
    const int kb = n3 * part / s.parts, ke = n3 * (part + 1) / s.parts;
    auto fetch_r = [&](int tile, int sl, double (&v)[4]) {
        const double* r = h.R + (long)min(tile * 16 + l16, h.Dxr - 1) * s.K3;
        const int k0 = sl * 16 + 4 * kg;
        if (sl * 16 + 16 <= s.K3) {
            const d2u_t x = *reinterpret_cast<const d2u_t*>(r + k0), z = *reinterpret_cast<const d2u_t*>(r + k0 + 2);
            v[0] = x.x; v[1] = x.y; v[2] = z.x; v[3] = z.y;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = k0 + q < s.K3 ? r[k0 + q] : 0.0;
        }
    };
    double rb[2][4];
    if (tile0 < t3 && kb < ke) fetch_r(tile0, kb, rb[0]);
    if (tile0 < t3 && kb + 1 < ke) fetch_r(tile0, kb + 1, rb[1]);

    // L's rows with zeros behind them, X3's padding, the matrix
    for (int r = wave; r < m1; r += NW)
        for (int k = lane; k < k1; k += 64)
            Ls[r * s.ldl + k] = k < h.Dyl ? h.L[((long)a0 * h.w0 + r) * h.Dyl + k] : 0.0;
    if (lane < k3 - s.K3)
        for (int r = wave; r < 16; r += NW) x3[r * s.ldx3 + s.K3 + lane] = 0.0;
    for (int e = t; e < h.nnz; e += NT) {
        sval[e] = h.val[e];
        scol[e] = h.col[e] * h.Dyr;
    }
    for (int o = t; o <= s.O; o += NT) srow[o] = h.rowptr[o];
    for (int o = t; o < s.O; o += NT) soff[o] = (o / h.w2) * s.ldx3 + (o % h.w2) * h.Dyr;
    __syncthreads();

    // X1
    for (int tile = wave; tile < t1; tile += NW) {
        const double* a = &Ls[min(l16, m1 - 1) * s.ldl + 4 * kg];
        d4_t acc = {0, 0, 0, 0};
        for (int sl = 0; sl < n1; ++sl, a += 16) {
            const double x[4] = {b[0][0], b[0][1], b[0][2], b[0][3]};
#pragma unroll
            for (int q = 0; q < 4; ++q) b[0][q] = b[1][q];
            if (ftile < t1) fetch(b[1]);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], x[q], acc, 0, 0, 0);
        }
        const int n = tile * 16 + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * r + kg < m1 && n < s.N1) x1[(4 * r + kg) * s.N1 + n] = acc[r];
    }
    __syncthreads();

    // the stage: an output o and column c for all rows a' at a time
    {
        const int all = s.O * h.Dyr, rows1 = s.I * h.Dyr, rows3 = h.dd * s.ldx3;
        const float inv = 1.0f / (float)h.Dyr;
        for (int idx = t; idx < all; idx += NT) {
            int o = (int)((float)idx * inv), c = idx - o * h.Dyr;
            if (c < 0) {
                --o;
                c += h.Dyr;
            } else if (c >= h.Dyr) {
                ++o;
                c -= h.Dyr;
            }
            const int e0 = srow[o], e1 = srow[o + 1];
            double* out = x3 + soff[o] + c;
            for (int a = 0; a < ga; a += 4) {
                double v[4] = {0, 0, 0, 0};
                const double* in = x1 + a * rows1 + c;
                // four terms at a time, so that their reads overlap
                for (int e = e0; e < e1; e += 4) {
                    double w[4], x[4][4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool on = e + u < e1;
                        const int at = on ? e + u : e;
                        w[u] = on ? sval[at] : 0.0;
                        const double* from = in + scol[at];
#pragma unroll
                        for (int q = 0; q < 4; ++q) x[u][q] = on && a + q < ga ? from[q * rows1] : 0.0;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] += w[u] * x[u][q];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (a + q < ga) out[(a + q) * rows3] = v[q];
            }
        }
    }
    __syncthreads();

    const int m3 = ga * h.dd;
    const long y0 = (long)a0 * h.dd;
    auto store = [&](int row, int n, double sum) {
        if (row >= m3 || n >= h.Dxr) return;
        const long at = (y0 + row) * h.Dxr + n;
        double v = h.beta * sum;
        if (h.C) v += h.alpha * h.C[at];
        h.y[at] = v;
    };
    const double* xr = x3 + min(l16, m3 - 1) * s.ldx3 + 4 * kg;
    for (int tile = tile0; tile < t3; tile += NW) {
        if (tile != tile0) {
            if (kb < ke) fetch_r(tile, kb, rb[0]);
            if (kb + 1 < ke) fetch_r(tile, kb + 1, rb[1]);
        }
        d4_t acc = {0, 0, 0, 0};
        auto step = [&](int sl, double (&cur)[4]) {
            const double x[4] = {cur[0], cur[1], cur[2], cur[3]};
            if (sl + 2 < ke) fetch_r(tile, sl + 2, cur);
            const double* a = xr + sl * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], x[q], acc, 0, 0, 0);
        };
        for (int sl = kb; sl < ke; sl += 2) {
            step(sl, rb[0]);
            if (sl + 1 < ke) step(sl + 1, rb[1]);
        }
        if (s.parts == 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) store(4 * r + kg, tile * 16 + l16, acc[r]);
        } else {
            // (X1 is no longer read)
#pragma unroll
            for (int r = 0; r < 4; ++r) x1[(tile * s.parts + part) * 256 + r * 64 + lane] = acc[r];
        }
    }
    if (s.parts > 1) {
        __syncthreads();
        for (int e = t; e < t3 * 256; e += NT) {
            const double* p = x1 + (e >> 8) * s.parts * 256 + (e & 255);
            double v = p[0];
            for (int q = 1; q < s.parts; ++q) v += p[q * 256];
            const int r = (e >> 6) & 3, l = e & 63;
            store(4 * r + (l >> 4), (e >> 8) * 16 + (l & 15), v);
        }
    }
}

__global__ __launch_bounds__(NT) void heff_small_kernel(Desc h) {
    extern __shared__ double heff_lds[];
    heff_tile(h, blockIdx.x, heff_lds);
}

__global__ __launch_bounds__(NT) void heff_grouped_kernel(const Desc* __restrict__ desc,
                                                          const int* __restrict__ count) {
    extern __shared__ double heff_lds[];
    const int G = count[0], total = count[1];
    for (int u = blockIdx.x; u < total; u += gridDim.x) {
        const int g = unit_problem(u, G, [&](int q) { return desc[q].start; });
        const Desc h = desc[g];
        heff_tile(h, u - h.start, heff_lds);
        __syncthreads();   // the LDS is the next unit's
    }
}

int rows_of(const HeffSmall& h) { return std::min(16 / h.w0, 16 / h.dd); }

Desc desc_of(const HeffSmall& h, int start) {
    Desc d{};
    d.L = h.L; d.theta = h.theta; d.R = h.R; d.C = h.C; d.y = h.y;
    d.alpha = h.alpha; d.beta = h.beta;
    d.Dxl = h.Dxl; d.Dyl = h.Dyl; d.Dxr = h.Dxr; d.Dyr = h.Dyr;
    d.w0 = h.w0; d.w2 = h.w2; d.dd = h.dd;
    d.g = rows_of(h);
    d.rowptr = h.rowptr; d.col = h.col; d.val = h.val; d.nnz = h.nnz;
    d.start = start;
    d.s = shape_of(d.Dyl, d.Dxr, d.Dyr, d.w0, d.w2, d.dd, d.g, d.nnz);
    return d;
}

}  // namespace

// One row tile in both products, the LDS of the batched launch, and at most
// HEFF_STEPS matrix-core steps (64 cycles each, two wavefronts a SIMD) a
// wavefront: bond 32 at d 2 has 20 and gains, bond 48 56 and loses; at d 4 bond 16
// has 12, bond 24 36.
bool heff_small_ok(const HeffSmall& h) {
    if (h.w0 < 1 || h.w0 > 16 || h.dd < 1 || h.dd > 16 || h.nnz < 0) return false;
    const long t1 = ((long)h.dd * h.Dyr + 15) / 16, t3 = (h.Dxr + 15) / 16;
    const long n1 = (h.Dyl + 15) / 16, n3 = ((long)h.w2 * h.Dyr + 15) / 16;
    const long s1 = (t1 + NW - 1) / NW * n1 * 4;
    const long s3 = t3 >= NW ? (t3 + NW - 1) / NW * n3 * 4 : (n3 + NW / t3 - 1) / (NW / t3) * 4;
    if (s1 + s3 > HEFF_STEPS) return false;
    const Shape s = shape_of(h.Dyl, h.Dxr, h.Dyr, h.w0, h.w2, h.dd, rows_of(h), h.nnz);
    return (size_t)s.total * sizeof(double) <= LDS_MAX;
}

void heff_small(const HeffSmall& h, hipStream_t st) {
    const Desc d = desc_of(h, 0);
    hipLaunchKernelGGL(heff_small_kernel, dim3((h.Dxl + d.g - 1) / d.g), dim3(NT), (size_t)d.s.total * sizeof(double),
                       st, d);
    HIP_CHECK(hipGetLastError());
}

size_t heff_desc_bytes() { return sizeof(Desc); }
int heff_desc_fill(const HeffSmall& h, int start, void* out) {
    const Desc d = desc_of(h, start);
    std::memcpy(out, &d, sizeof(d));
    return (h.Dxl + d.g - 1) / d.g;
}
void heff_grouped(const void* desc, const int* count, hipStream_t s) {
    hipLaunchKernelGGL(heff_grouped_kernel, dim3(256), dim3(NT), LDS_MAX, s, static_cast<const Desc*>(desc), count);
    HIP_CHECK(hipGetLastError());
}

}  // namespace ite
