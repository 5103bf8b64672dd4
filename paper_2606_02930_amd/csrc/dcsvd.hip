// Singular value decomposition of an upper bidiagonal matrix by divide and
// conquer (Gu and Eisenstat, "A divide-and-conquer algorithm for the
// bidiagonal SVD", SIAM J. Matrix Anal. Appl. 16, 1995).
//
// A node is a range [a, b) of rows with the columns [a, b] (without column n
// at the right end).  Its middle row m = a + (b - a) / 2 holds alpha = d_m in
// column m and beta = e_m in column m + 1; the rows before and after m are its
// children.  With the children's singular values and vectors, and their null
// vectors (a child has one column more than rows), the node's matrix becomes
// orthogonally equivalent to diag(0, d) with a first row z.  Entries with a
// small |z_j| (deflation_limit), and all but one of a group of equal
// d_j (after a rotation that leaves one of their z_j), are singular values as
// they stand (deflation).  The other singular values are the roots of
//   1 + sum_j z_j^2 / (d_j^2 - sigma^2) = 0,
// one between each two poles, found as the distance x = sigma^2 - d_c^2 from
// the nearer pole, so that every difference d_j^2 - sigma^2 =
// (d_j - d_c)(d_j + d_c) - x keeps its relative accuracy.  z is then
// recomputed from the roots (the vectors of a matrix that has exactly these
// singular values are orthogonal to rounding), the vectors follow in closed
// form, and one product with the children's vectors finishes the node.
//
// Vectors are rows: UT, VT [n][n].  The null vector of node [a, b) is row b of
// VT.  Subtrees of at most LEAF rows are done by one workgroup in LDS, down to
// single rows; a level above takes five launches for all its nodes:
// dc_prep (sort, deflation), dc_roots (roots; the children's vectors gathered
// in the order of the poles, deflated ones to their final place), dc_zhat,
// dc_small_vectors and dc_gemm.  Everything is FP64 and every reduction has a
// fixed order.
#include "gemm_tile.h"
#include "internal.h"
#include "wave.h"

#include <algorithm>

namespace ite {
namespace {

constexpr int LEAF = 32;
constexpr double EPS = 2.220446049250313e-16;

// What counts as zero, and as equal, at a value d of a node with norm nrm: 8 eps
// of the norm at the norm itself, where that saves work on equal values, falling
// to eps for small d.  (With 8 eps throughout a vanishing value came back as
// 1.8e-15 of the largest and values up to that as zero, so that a cutoff of 1e-30
// kept 6 to 9 vectors of a block of rank 3; with eps throughout a block of equal
// values of 33 rows took 208 us instead of 130.)
//
// Never below FLOOR, so that the squares of what is left, and what is divided by
// them, stay numbers (the matrix is scaled to a largest entry of one).
constexpr double FLOOR = 1e-120;
__device__ inline double deflation_limit(double nrm, double d) { return fmax(EPS * fma(7.0, d, nrm), FLOOR); }
// The one singular value left of a node.
__device__ inline double lone_value(double z) { return fabs(z) > FLOOR ? fabs(z) : 0.0; }

struct Node {
    int a, m, b;
};
// Node q of a depth (bit i of q from the top: right child).
__device__ inline Node node_at(int a, int b, int depth, int q) {
    for (int i = depth - 1; i >= 0; --i) {
        const int m = a + (b - a) / 2;
        if ((q >> i) & 1) a = m + 1;
        else b = m;
    }
    return Node{a, a + (b - a) / 2, b};
}
// The node of a depth that holds row g; q = -1 when g is a middle row above.
__device__ inline Node node_of(int n, int depth, int g, int& q) {
    int a = 0, b = n;
    q = 0;
    for (int i = 0; i < depth; ++i) {
        const int m = a + (b - a) / 2;
        if (g == m) {
            q = -1;
            return Node{0, 0, 0};
        }
        q *= 2;
        if (g > m) {
            a = m + 1;
            ++q;
        } else {
            b = m;
        }
    }
    return Node{a, a + (b - a) / 2, b};
}

// NaN as zero, so that orders and counts stay those of a finite matrix (the
// scale, and with it every singular value, is NaN where an entry is not finite).
__device__ inline double clean(double v) { return v == v ? v : 0.0; }

// r = sqrt(x^2 + y^2), c = x / r, s = y / r for values scaled to at most about 1
// (both below 1e-150: as zeros).
__device__ inline void plane_rotation(double x, double y, double& r, double& c, double& s) {
    const double q = x * x + y * y;
    if (q > 1e-300) {
        const double i = recip_sqrt(q);
        c = x * i;
        s = y * i;
        r = q * i;
    } else {
        c = 1.0;
        s = 0.0;
        r = q == q ? 0.0 : q;
    }
}

// One Newton step: a relative error of about 1e-14, for the steps of an
// iteration that checks its own result.
__device__ inline double quick_recip(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r, 1.0), r, r);
}
__device__ inline double quick_rsqrt(double x) {
    const double r = __builtin_amdgcn_rsq(x);
    return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// One update of a root of f(x) = 1 + psi(x) + phi(x): psi (the poles up to
// da = pole - x) and phi (those from db on) are replaced by r + s / (pole - x)
// with their values and slopes at x (Bunch, Nielsen and Sorensen); kept inside
// the bracket.  Returns true when x is the root to rounding.
__device__ inline bool root_step(double& x, double& lo, double& hi, double psi, double dpsi, double phi, double dphi,
                                 double da, double db, bool last) {
    const double f = 1.0 + psi + phi;
    if (f < 0.0) lo = x;
    else hi = x;
    if (!(fabs(f) > 8.0 * EPS * (1.0 - psi + phi))) return true;
    double eta;
    const double s = dpsi * da * da;
    if (last) {
        eta = da + s * quick_recip(1.0 + (psi - dpsi * da));
    } else {
        const double tt = dphi * db * db;
        const double cc = 1.0 + (psi - dpsi * da) + (phi - dphi * db);
        const double A = cc * (da + db) + s + tt, B = da * db * f;
        const double q = fmax(A * A - 4.0 * cc * B, 1e-300), disc = q * quick_rsqrt(q);
        eta = A > 0.0 ? 2.0 * B * quick_recip(A + disc) : (A - disc) * quick_recip(2.0 * cc);
    }
    double xn = x + eta;
    if (!(xn > lo && xn < hi)) xn = 0.5 * (lo + hi);
    const bool done = xn == x || fabs(hi - lo) <= EPS * fabs(xn);
    x = xn;
    return done;
}
constexpr int ROOT_ITERS = 100;

// Start of a root between the poles di < di1 from f at the middle of their
// squares: the nearer pole dc, the bracket, and the root with the other poles'
// sum held at its value there.
__device__ inline void first_root(double f, double mid, double zi2, double zn2, double di, double di1, double& x,
                                  double& lo, double& hi, double& dc) {
    // at the middle the two poles' terms are -zi2 / mid and zn2 / mid
    const double im = quick_recip(mid), cc = f + (zi2 - zn2) * im;
    const bool left = f >= 0.0;
    dc = left ? di : di1;
    lo = left ? 0.0 : -mid;
    hi = left ? mid : 0.0;
    const double p0 = left ? 0.0 : -2.0 * mid, p1 = left ? 2.0 * mid : 0.0;
    const double A = cc * (p0 + p1) + zi2 + zn2, B = zi2 * p1 + zn2 * p0;
    const double q = fmax(A * A - 4.0 * cc * B, 1e-300), disc = q * quick_rsqrt(q);
    x = A > 0.0 ? 2.0 * B * quick_recip(A + disc) : (A - disc) * quick_recip(2.0 * cc);
    if (!(x > lo && x < hi)) x = left ? mid : -mid;
}

// sigma from its pole and distance.
__device__ inline double sigma_of(double dc, double x) {
    const double s2 = dc * dc + x;
    return s2 > 0.0 ? dc + x / (dc + sqrt(s2)) : dc;
}

// ---------------------------------------------------------------------------
// Subtrees in LDS
// ---------------------------------------------------------------------------

// A level of a subtree in three steps: a wavefront a node sorts and deflates;
// eight lanes a row find the roots, recompute z and form the vectors, four poles
// a lane (one wavefront a SIMD: more would only wait for each other's issue
// slots); eight wavefronts multiply.  Every row of the level is a row of one
// LEAF x LEAF matrix of weights: the small vectors of its node, or a one for a
// deflated row or a null vector, against source rows gathered by `src`.
constexpr int LNT = 1024;
constexpr int LNW = LNT / 64;

struct LeafLDS {
    double U[2][LEAF][LEAF + 1], V[2][LEAF + 1][LEAF + 2];
    double Us[LEAF][LEAF + 1], Vs[LEAF][LEAF + 1];
    double sg[2][LEAF + 1], d[LEAF], e[LEAF];
    // a node's entries from its first row on: the order (scratch of its
    // wavefront), then poles, z and z recomputed
    double sd[LEAF], sz[LEAF], cr[LEAF], sr[LEAF], dd[LEAF], zz[LEAF], zh[LEAF], x[LEAF], dc[LEAF];
    int srow[LEAF], prev[LEAF];
    int src[LEAF];                 // source row of column c of the weights
    int kind[LEAF], na[LEAF], nk[LEAF];
    int lasta;                     // first row of the node whose null vector is row LEAF
    double red[LNW];
};
enum { ROW_PRODUCT = 0, ROW_COPY = 1, ROW_NULL = 2 };

__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// Sort and deflation of one node of a subtree by one wavefront (local rows, at
// most 32).  `null`: column b exists.
__device__ __forceinline__ void leaf_deflate(LeafLDS& L, int cur, int a, int m, int b, bool null,
                                             int lane) {
    const int N = b - a;
    auto& U = L.U[cur];
    auto& V = L.V[cur];
    if (lane == 0 && null) {
        if (b < LEAF) {
            L.kind[b] = ROW_NULL;
            L.src[b] = b;
        } else {
            L.lasta = a;
        }
    }
    if (N == 0) {
        if (null && lane <= LEAF) V[b][lane] = lane == b ? 1.0 : 0.0;
        return;
    }
    if (lane < N) {
        L.na[a + lane] = a;
        L.kind[a + lane] = ROW_COPY;
        L.nk[a + lane] = 0;
    }
    const double alpha = L.d[m], beta = L.e[m];
    if (N == 1) {
        double r = fabs(alpha), c = alpha < 0.0 ? -1.0 : 1.0, s = 0.0;
        if (null) plane_rotation(alpha, beta, r, c, s);
        if (lane == 0) {
            U[a][a] = 1.0;
            V[a][a] = c;
            if (null) {
                V[a][b] = s;
                V[b][a] = -s;
                V[b][b] = c;
            }
            L.sg[cur ^ 1][a] = clean(r);
            L.src[a] = a;
        }
        return;
    }
    const double x0 = alpha * V[m][m], y0 = null ? beta * V[b][m + 1] : 0.0;
    double r0 = x0, c0 = 1.0, s0 = 0.0;
    if (null) plane_rotation(x0, y0, r0, c0, s0);
    double zv = 0.0, dv = 0.0;
    if (lane < N) {
        const int r = a + lane;
        dv = r == m ? 0.0 : clean(L.sg[cur][r]);
        zv = clean(r < m ? alpha * V[r][m] : (r > m ? beta * V[r][m + 1] : r0));
    }
    wave_fence();
    if (lane <= N && null) {
        const int c = a + lane;
        const double w1 = V[m][c], w2 = V[b][c];
        V[m][c] = c0 * w1 + s0 * w2;
        V[b][c] = c0 * w2 - s0 * w1;
    }
    double* sd = L.sd + a;
    double* sz = L.sz + a;
    int* srow = L.srow + a;
    if (lane < N) {
        U[m][a + lane] = a + lane == m ? 1.0 : 0.0;
    }
    const double nrm = fmax(wave_max_nonneg(dv), fmax(fabs(clean(alpha)), fabs(clean(beta))));
    const double tol = deflation_limit(nrm, 0.0);
    wave_fence();
    const int lm = m - a;
    int rank = lane == lm ? 0 : 1;
    for (int t = 0; t < N; ++t) {
        const double k = lane_value(dv, t);
        if (lane != lm && t != lm) rank += k < dv || (k == dv && t < lane);
    }
    if (lane < N) {
        sd[rank] = dv;
        sz[rank] = zv;
        srow[rank] = a + lane;
    }
    wave_fence();
    double ds = 0.0, zs = 0.0;
    int act = 1, row = 0;
    if (lane < N) {
        ds = sd[lane];
        zs = sz[lane];
        row = srow[lane];
        if (lane == 0 && !(fabs(zs) > tol)) zs = zs < 0.0 ? -tol : tol;
    }
    const double lim = deflation_limit(nrm, ds);
    const bool surv = lane > 0 && lane < N && fabs(zs) > lim;
    const bool tiny = surv && ds <= tol;
    const unsigned long long below = (1ull << lane) - 1;
    const unsigned long long ms = __ballot(surv && !tiny);
    int pv = -1;
    if (surv && !tiny) {
        const unsigned long long q = ms & below;
        pv = q ? 63 - __clzll(q) : -1;
        act = pv >= 0 && ds - sd[pv] <= lim ? 2 : 0;
    } else if (tiny) {
        act = 3;
    } else if (lane == 0) {
        act = 0;
    }
    const bool in = lane < N;
    const unsigned long long m0 = __ballot(in && act == 0), m2 = __ballot(in && act == 2), m3 = __ballot(in && act == 3);
    const int K = __popcll(m0);
    const int slot = __popcll(m0 & below);
    if (in) {
        sz[lane] = zs;
        if (act == 0) {
            // the chain that starts here: its rows rotate into one
            double z = zs, dl = ds;
            int last = row;
            if (lane == 0) {
                for (unsigned long long q = m3; q; q &= q - 1) {
                    const int t = __ffsll((long long)q) - 1;
                    plane_rotation(z, sz[t], z, L.cr[a + t], L.sr[a + t]);
                }
            } else if (m2) {
                const unsigned long long later = ms & ~below & ~(1ull << lane);
                for (unsigned long long q = later; q; q &= q - 1) {
                    const int t = __ffsll((long long)q) - 1;
                    if (!((m2 >> t) & 1)) break;
                    plane_rotation(sz[t], z, z, L.cr[a + t], L.sr[a + t]);
                    dl = sd[t];
                    last = srow[t];
                }
            }
            L.dd[a + slot] = dl;
            L.zz[a + slot] = z;
            L.src[a + slot] = last;
            L.kind[a + slot] = ROW_PRODUCT;
        } else {
            const int o = a + K + (lane - slot);      // lane - slot deflated entries before this one
            L.src[o] = act == 2 ? srow[pv] : row;
            L.sg[cur ^ 1][o] = act == 2 ? sd[pv] : (act == 3 ? 0.0 : ds);
        }
        L.prev[a + lane] = pv;
        L.nk[a + lane] = K;
    }
    wave_fence();
    for (unsigned long long q = m2 | m3; q; q &= q - 1) {
        const int t = __ffsll((long long)q) - 1;
        const double c = L.cr[a + t], s = L.sr[a + t];
        const int rt = srow[t];
        if ((m3 >> t) & 1) {
            if (lane <= N) {
                const double x = V[m][a + lane], y = V[rt][a + lane];
                V[m][a + lane] = c * x + s * y;
                V[rt][a + lane] = c * y - s * x;
            }
        } else {
            const int rp = srow[L.prev[a + t]];
            if (lane <= N) {
                const double x = V[rp][a + lane], y = V[rt][a + lane];
                V[rp][a + lane] = c * x - s * y;
                V[rt][a + lane] = s * x + c * y;
            }
            if (lane < N) {
                const double x = U[rp][a + lane], y = U[rt][a + lane];
                U[rp][a + lane] = c * x - s * y;
                U[rt][a + lane] = s * x + c * y;
            }
        }
        wave_fence();
    }
}

// Sums and products over groups of eight lanes, to all of them.
__device__ inline double sum8(double v) {
    v += dpp_move<0xB1, 0xf>(v);
    v += dpp_move<0x4E, 0xf>(v);
    return v + dpp_move<0x141, 0xf>(v);
}
__device__ inline double product8(double v) {
    v *= dpp_move<0xB1, 0xf>(v);
    v *= dpp_move<0x4E, 0xf>(v);
    return v * dpp_move<0x141, 0xf>(v);
}

// Roots, recomputed z and the rows of weights of a level whose nodes have at
// most 8 PL rows: row r (a root, then a pole, then a root again), poles j0,
// j0 + 8, ...
template <int PL>
__device__ __forceinline__ void leaf_vectors(LeafLDS& L, int cur, int len, int rows) {
    const int t = threadIdx.x, r = t >> 3, j0 = t & 7;
    const bool mine = t < 8 * LEAF && r < len && L.kind[r] == ROW_PRODUCT;
    const int a = mine ? L.na[r] : 0, K = mine ? L.nk[r] : 0, i = r - a;
    double dj[PL], z[PL], x = 0.0, dc = 0.0;
    if (mine) {
#pragma unroll
        for (int q = 0; q < PL; ++q) {
            const int j = j0 + 8 * q;
            dj[q] = j < K ? L.dd[a + j] : 0.0;
            z[q] = j < K ? L.zz[a + j] : 0.0;
        }
        if (K > 1) {
            const bool last = i == K - 1;
            const double di = L.dd[a + i], di1 = last ? 0.0 : L.dd[a + i + 1];
            // poles up to i and after i by factors of one and zero
            double z2[PL], del[PL], lower[PL], upper[PL];
#pragma unroll
            for (int q = 0; q < PL; ++q) {
                z2[q] = z[q] * z[q];
                lower[q] = j0 + 8 * q <= i ? 1.0 : 0.0;
                upper[q] = 1.0 - lower[q];
            }
            double lo = 0.0, hi;
            dc = di;
            if (last) {
                double tot = z2[0];
#pragma unroll
                for (int q = 1; q < PL; ++q) tot += z2[q];
                hi = sum8(tot) * (1.0 + 8.0 * EPS);
                x = 0.5 * hi;
            } else {
                const double mid = 0.5 * (di1 - di) * (di1 + di), zi = L.zz[a + i], zn = L.zz[a + i + 1];
                double f = 0.0;
#pragma unroll
                for (int q = 0; q < PL; ++q)
                    f += z2[q] * recip(j0 + 8 * q < K ? (dj[q] - di) * (dj[q] + di) - mid : 1.0);
                first_root(1.0 + sum8(f), mid, zi * zi, zn * zn, di, di1, x, lo, hi, dc);
            }
#pragma unroll
            for (int q = 0; q < PL; ++q) del[q] = j0 + 8 * q < K ? (dj[q] - dc) * (dj[q] + dc) : 1e100;
            const double da0 = (di - dc) * (di + dc), db0 = last ? 0.0 : (di1 - dc) * (di1 + dc);
            for (int it = 0; it < ROOT_ITERS; ++it) {
                double psi = 0.0, dpsi = 0.0, phi = 0.0, dphi = 0.0;
#pragma unroll
                for (int q = 0; q < PL; ++q) {
                    const double rc = recip(del[q] - x), tt = z2[q] * rc, t2 = tt * rc;
                    psi = fma(tt, lower[q], psi);
                    dpsi = fma(t2, lower[q], dpsi);
                    phi = fma(tt, upper[q], phi);
                    dphi = fma(t2, upper[q], dphi);
                }
                if (root_step(x, lo, hi, sum8(psi), sum8(dpsi), sum8(phi), sum8(dphi), da0 - x,
                              last ? 0.0 : db0 - x, last))
                    break;
            }
            if (j0 == 0) {
                L.sg[cur ^ 1][r] = sigma_of(dc, x);
                L.x[r] = x;
                L.dc[r] = dc;
            }
        } else if (j0 == 0) {
            L.sg[cur ^ 1][r] = lone_value(z[0]);
        }
    }
    __syncthreads();
    if (mine && K > 1) {
        // z of pole i from the roots
        const double di = L.dd[a + i];
        double f = 1.0;
#pragma unroll
        for (int q = 0; q < PL; ++q) {
            const int j = j0 + 8 * q;
            if (j >= K) continue;
            f *= L.x[a + j] - (di - L.dc[a + j]) * (di + L.dc[a + j]);
            if (j < K - 1) {
                const double o = j < i ? dj[q] : L.dd[a + j + 1];
                f *= recip((o - di) * (o + di));
            }
        }
        f = sqrt(fabs(product8(f)));
        if (j0 == 0) L.zh[r] = L.zz[r] < 0.0 ? -f : f;
    }
    __syncthreads();
    if (t < 8 * LEAF) {
        double u[PL], v[PL], nu = 0.0, nv = 0.0;
#pragma unroll
        for (int q = 0; q < PL; ++q) {
            const int j = j0 + 8 * q;
            u[q] = v[q] = 0.0;
            if (!mine || j >= K) continue;
            v[q] = K > 1 ? L.zh[a + j] * recip((dj[q] - dc) * (dj[q] + dc) - x) : (z[0] < 0.0 ? -1.0 : 1.0);
            u[q] = K > 1 ? (j == 0 ? -1.0 : dj[q] * v[q]) : 1.0;
            nu += u[q] * u[q];
            nv += v[q] * v[q];
        }
        nu = recip_sqrt(sum8(nu));
        nv = recip_sqrt(sum8(nv));
        // zero but for the node's poles, or a one for the row itself
        const int kind = r < rows ? L.kind[r] : -1;
#pragma unroll
        for (int c = 0; c < LEAF; c += 8)
            if (!mine || c + j0 < a || c + j0 >= a + K) {
                L.Us[r][c + j0] = kind == ROW_COPY && c + j0 == r ? 1.0 : 0.0;
                L.Vs[r][c + j0] = (kind == ROW_COPY || kind == ROW_NULL) && c + j0 == r ? 1.0 : 0.0;
            }
#pragma unroll
        for (int q = 0; q < PL; ++q) {
            const int j = j0 + 8 * q;
            if (mine && j < K) {
                L.Us[r][a + j] = u[q] * nu;
                L.Vs[r][a + j] = v[q] * nv;
            }
        }
    }
    __syncthreads();
}

// A power of two near the largest |d|, |e| (2^-1000 at least).
__device__ inline double pow2_scale(double mx, bool inverse) {
    if (!(mx > 0.0) || !(mx < 1e300)) return 1.0;
    int ex;
    (void)frexp(mx, &ex);
    ex = max(ex, -1000);
    return ldexp(1.0, inverse ? -ex : ex);
}

__global__ __launch_bounds__(LNT) void dc_leaf_kernel(DcWork w, int depth) {
    __shared__ LeafLDS L;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, n = w.n;
    double mx = 0.0;       // infinite for entries that are not finite (fmax passes NaN by)
    for (int i = t; i < n; i += LNT) {
        const double d = fabs(w.d[i]), e = i + 1 < n ? fabs(w.e[i]) : 0.0;
        mx = d < INFINITY && e < INFINITY ? fmax(mx, fmax(d, e)) : INFINITY;
    }
    mx = wave_max_nonneg(mx);
    if (lane == 0) L.red[wv] = mx;
    __syncthreads();
    mx = L.red[0];
    for (int q = 1; q < LNW; ++q) mx = fmax(mx, L.red[q]);
    const double inv = pow2_scale(mx, true);
    if (blockIdx.x == 0 && t == 0) {
        *w.scale = mx < INFINITY ? pow2_scale(mx, false) : NAN;
        *w.inv = inv;
    }
    const Node root = node_at(0, n, depth, blockIdx.x);
    const int a0 = root.a, len = root.b - root.a;
    if (t < LEAF) {
        L.kind[t] = ROW_COPY;      // (rows past the subtree's)
        L.src[t] = 0;
    }
    if (t < len) {
        L.d[t] = w.d[a0 + t] * inv;
        L.e[t] = a0 + t + 1 < n ? w.e[a0 + t] * inv : 0.0;
    }
    for (int x = t; x < 2 * LEAF * (LEAF + 1); x += LNT) (&L.U[0][0][0])[x] = 0.0;
    for (int x = t; x < 2 * (LEAF + 1) * (LEAF + 2); x += LNT) (&L.V[0][0][0])[x] = 0.0;
    __syncthreads();
    const int rows = min(LEAF, len + (a0 + len < n));      // with the subtree's null vector
    int top = 0;
    for (int sz = len; sz > 1; sz /= 2) ++top;
    int cur = 0;
    for (int lv = top; lv >= 0; --lv) {
        for (int q = wv; q < (1 << lv); q += LNW) {
            const Node nd = node_at(0, len, lv, q);
            leaf_deflate(L, cur, nd.a, nd.m, nd.b, a0 + nd.b < n, lane);
        }
        __syncthreads();
        if ((len >> lv) <= 8) leaf_vectors<1>(L, cur, len, rows);
        else if ((len >> lv) <= 16) leaf_vectors<2>(L, cur, len, rows);
        else leaf_vectors<LEAF / 8>(L, cur, len, rows);
        // the products: a 16 x 16 tile of U or V a wavefront; column LEAF of V and
        // the subtree's null vector by others
        if (wv < 8) {
            const int side = wv >> 2, r0 = 16 * ((wv >> 1) & 1), c0 = 16 * (wv & 1), l16 = lane & 15, kg = lane >> 4;
            if (r0 < rows && c0 < len + 1) {
                d4_t acc = {0, 0, 0, 0};
#pragma unroll
                for (int k = 0; k < LEAF; k += 4) {
                    const int g = L.src[k + kg];
                    const double wt = side ? L.Vs[r0 + l16][k + kg] : L.Us[r0 + l16][k + kg];
                    const double y = side ? L.V[cur][g][c0 + l16] : L.U[cur][g][c0 + l16];
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(wt, y, acc, 0, 0, 0);
                }
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const int row = r0 + 4 * rr + kg;
                    if (side) L.V[cur ^ 1][row][c0 + l16] = acc[rr];
                    else L.U[cur ^ 1][row][c0 + l16] = acc[rr];
                }
            }
        } else if (wv < 12) {
            const int rr = (t - 512) >> 3, j0 = t & 7;
            double v = 0.0;
#pragma unroll
            for (int c = j0; c < LEAF; c += 8) v += L.Vs[rr][c] * L.V[cur][L.src[c]][LEAF];
            v = sum8(v);
            if (j0 == 0 && len == LEAF) L.V[cur ^ 1][rr][LEAF] = v;
        } else if (wv == 12 && len == LEAF && a0 + len < n && lane <= len) {
            L.V[cur ^ 1][len][lane] = lane >= L.lasta ? L.V[cur][len][lane] : 0.0;
        }
        __syncthreads();
        cur ^= 1;
    }
    for (int x = t; x < (len + 1) * (len + 1); x += LNT) {
        const int r = x / (len + 1), c = x % (len + 1);
        if (a0 + r >= n || a0 + c >= n) continue;
        const long at = (long)(a0 + r) * n + a0 + c;
        if (r < len && c < len) w.UT[0][at] = L.U[cur][r][c];
        w.VT[0][at] = L.V[cur][r][c];
    }
    if (t < len) w.sg[0][a0 + t] = L.sg[cur][t];
}

// ---------------------------------------------------------------------------
// Levels above the subtrees
// ---------------------------------------------------------------------------

constexpr int PREP_CAP = 2048;      // rows of a node kept in LDS

// Entry s of a node's order (ascending d, the middle row first): act 0 starts
// an undeflated vector, 1 is deflated as it stands, 2 rotates with the entry
// before it in its chain, 3 with the middle row (right vectors only).
template <int PREP_NT>
__global__ __launch_bounds__(PREP_NT) void dc_prep_kernel(DcWork w, int depth, int cur) {
    __shared__ double lkey[PREP_CAP], lsd[PREP_CAP], lsz[PREP_CAP];
    __shared__ int lrow[PREP_CAP], lact[PREP_CAP], lcl[PREP_CAP];
    __shared__ double red[PREP_NT / 64];
    __shared__ int cnt[PREP_NT / 64];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, n = w.n;
    const Node nd = node_at(0, n, depth, blockIdx.x);
    const int a = nd.a, m = nd.m, b = nd.b, N = b - a;
    const bool small = N <= PREP_CAP;
    double* key = small ? lkey : w.t0 + a;
    double* sd = small ? lsd : w.t1 + a;
    double* sz = small ? lsz : w.t2 + a;
    int* row = w.ord + a;
    int* act = small ? lact : w.i0 + a;
    int* cl = small ? lcl : w.i1 + a;
    int* srow = small ? lrow : row;
    const double* VT = w.VT[cur];
    const double* sg = w.sg[cur];
    double* sgo = w.sg[cur ^ 1];
    const double inv = *w.inv;
    const double alpha = clean(w.d[m] * inv), beta = m + 1 < n ? clean(w.e[m] * inv) : 0.0;
    const bool null = b < n;
    double r0 = alpha * clean(VT[(long)m * n + m]), c0 = 1.0, s0 = 0.0;
    if (null) plane_rotation(r0, beta * clean(VT[(long)b * n + m + 1]), r0, c0, s0);
    double mx = 0.0;
    for (int i = t; i < N; i += PREP_NT) {
        const double v = a + i == m ? 0.0 : clean(sg[a + i]);
        key[i] = v;
        mx = fmax(mx, v);
    }
    mx = wave_max_nonneg(mx);
    if (lane == 0) red[wv] = mx;
    __syncthreads();
    for (int q = 0; q < PREP_NT / 64; ++q) mx = fmax(mx, red[q]);
    const double nrm = fmax(mx, fmax(fabs(alpha), fabs(beta))), tol = deflation_limit(nrm, 0.0);
    // ascending order, the middle row first: a bitonic network over the keys in
    // LDS (row numbers break ties; pairs up to 64 apart stay in a wavefront)
    auto zof = [&](int r) {
        if (r == m) return fabs(r0) > tol ? r0 : (r0 < 0.0 ? -tol : tol);
        return clean(r < m ? alpha * VT[(long)r * n + m] : beta * VT[(long)r * n + m + 1]);
    };
    if (small) {
        int n2 = 2;
        while (n2 < N) n2 *= 2;
        for (int i = t; i < n2; i += PREP_NT) {
            lrow[i] = i;
            if (i >= N) key[i] = INFINITY;
            else if (a + i == m) key[i] = -1.0;
        }
        __syncthreads();
        for (int k = 2; k <= n2; k *= 2)
            for (int h = k / 2; h > 0; h /= 2) {
                if (h > 64) __syncthreads();
                for (int p = t; p < n2 / 2; p += PREP_NT) {
                    const int i = 2 * p - (p & (h - 1)), q = i + h;
                    const double x = key[i], y = key[q];
                    const int rx = lrow[i], rq = lrow[q];
                    const bool up = (i & k) == 0, gt = x > y || (x == y && rx > rq);
                    if (gt == up) {
                        key[i] = y;
                        key[q] = x;
                        lrow[i] = rq;
                        lrow[q] = rx;
                    }
                }
                if (h > 64) __syncthreads();
                else wave_fence();
            }
        __syncthreads();
        for (int i = t; i < N; i += PREP_NT) {
            const int r = a + lrow[i];
            sd[i] = fmax(key[i], 0.0);
            sz[i] = zof(r);
            lrow[i] = r;
        }
    } else {
        for (int i = t; i < N; i += PREP_NT) {
            const int r = a + i;
            const double v = key[i];
            int rank = 0;
            if (r != m) {
                for (int q = 0; q < N; ++q) rank += key[q] < v || (key[q] == v && q < i);
                if (v == 0.0 && i < m - a) ++rank;      // the middle row (key 0) comes first whatever ties with it
            }
            sd[rank] = v;
            sz[rank] = zof(r);
            srow[rank] = r;
        }
    }
    __syncthreads();
    // survivors with d above the tolerance, compacted in order
    int total = 0;
    for (int base = 0; base < N; base += PREP_NT) {
        const int s = base + t;
        const bool surv = s > 0 && s < N && fabs(sz[s]) > deflation_limit(nrm, sd[s]), tiny = surv && sd[s] <= tol;
        if (s < N) act[s] = tiny ? 3 : (s == 0 ? 0 : 1);
        const unsigned long long bal = __ballot(surv && !tiny);
        if (lane == 0) cnt[wv] = __popcll(bal);
        __syncthreads();
        int before = total;
        for (int q = 0; q < wv; ++q) before += cnt[q];
        if (surv && !tiny) cl[before + __popcll(bal & ((1ull << lane) - 1))] = s;
        for (int q = 0; q < PREP_NT / 64; ++q) total += cnt[q];
        __syncthreads();
    }
    for (int ci = t; ci < total; ci += PREP_NT) {
        const int s = cl[ci];
        act[s] = ci > 0 && sd[s] - sd[cl[ci - 1]] <= deflation_limit(nrm, sd[s]) ? 2 : 0;
    }
    __syncthreads();
    // destinations: starts by their order, then the deflated entries
    int K = 0;
    for (int base = 0; base < N; base += PREP_NT) {
        const int s = base + t;
        const unsigned long long bal = __ballot(s < N && act[s] == 0);
        if (lane == 0) cnt[wv] = __popcll(bal);
        __syncthreads();
        int before = K;
        for (int q = 0; q < wv; ++q) before += cnt[q];
        if (s < N) {
            const int starts = before + __popcll(bal & ((1ull << lane) - 1));
            w.dst[a + s] = act[s] == 0 ? starts : s - starts;     // + K below for the deflated
            w.act[a + s] = act[s];
            w.nxt[a + s] = -1;
            if (small) row[s] = srow[s];
        }
        for (int q = 0; q < PREP_NT / 64; ++q) K += cnt[q];
        __syncthreads();
    }
    for (int s = t; s < N; s += PREP_NT) {
        if (act[s] == 0) continue;
        const int o = w.dst[a + s] + K;
        w.dst[a + s] = o;
        if (act[s] != 2) sgo[a + o] = act[s] == 3 ? 0.0 : sd[s];
    }
    __syncthreads();
    // chains: z accumulates along them, the values before the last deflate
    auto rotate = [&](int prev, int s, double& z, bool mid) {
        double c, q;
        plane_rotation(z, sz[s], z, c, q);
        w.cr[a + s] = mid ? c : q;
        w.sr[a + s] = mid ? q : c;
        w.nxt[a + prev] = s;
    };
    if (t == 0) {
        double z = sz[0];
        int prev = 0;
        for (int s = 1; s < N && sd[s] <= tol; ++s)
            if (act[s] == 3) {
                rotate(prev, s, z, true);
                prev = s;
            }
        w.dd[a] = 0.0;
        w.zz[a] = z;
        w.K[blockIdx.x] = K;
        w.cs[2 * blockIdx.x] = c0;
        w.cs[2 * blockIdx.x + 1] = s0;
    }
    for (int ci = t; ci < total; ci += PREP_NT) {
        const int s = cl[ci];
        if (act[s] != 0) continue;
        double z = sz[s], dl = sd[s];
        int prev = s;
        for (int k = ci + 1; k < total && act[cl[k]] == 2; ++k) {
            const int u = cl[k];
            sgo[a + w.dst[a + u]] = dl;
            rotate(prev, u, z, false);
            dl = sd[u];
            prev = u;
        }
        w.dd[a + w.dst[a + s]] = dl;
        w.zz[a + w.dst[a + s]] = z;
    }
}

// The first ceil(n / 4) workgroups find the roots (a wavefront each); the
// others gather the children's vectors: an order entry and 256 columns each,
// nch workgroups an entry.
__global__ __launch_bounds__(256) void dc_roots_kernel(DcWork w, int depth, int cur, int nch) {
    const int n = w.n, lane = threadIdx.x & 63, nroot = (n + 3) / 4;
    int q;
    if ((int)blockIdx.x < nroot) {
        const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
        if (g >= n) return;
        const Node nd = node_of(n, depth, g, q);
        if (q < 0) return;
        const int K = w.K[q], i = g - nd.a;
        if (i >= K) return;
        const double* __restrict__ dd = w.dd + nd.a;
        const double* __restrict__ zz = w.zz + nd.a;
        double* sgo = w.sg[cur ^ 1];
        if (K == 1) {
            if (lane == 0) {
                sgo[g] = lone_value(zz[0]);
                w.x[g] = zz[0] * zz[0];
                w.dc[g] = 0.0;
            }
            return;
        }
        const bool last = i == K - 1;
        const double di = dd[i], di1 = last ? 0.0 : dd[i + 1];
        double lo = 0.0, hi, x, dc = di;
        if (last) {
            double tot = 0.0;
            for (int j = lane; j < K; j += 64) tot += zz[j] * zz[j];
            hi = wave_sum(tot) * (1.0 + 8.0 * EPS);
            x = 0.5 * hi;
        } else {
            const double mid = 0.5 * (di1 - di) * (di1 + di), zi = zz[i], zn = zz[i + 1];
            double f = 0.0;
            for (int j = lane; j < K; j += 64) f += zz[j] * zz[j] * recip((dd[j] - di) * (dd[j] + di) - mid);
            first_root(1.0 + wave_sum(f), mid, zi * zi, zn * zn, di, di1, x, lo, hi, dc);
        }
        for (int it = 0; it < ROOT_ITERS; ++it) {
            double psi = 0.0, dpsi = 0.0, phi = 0.0, dphi = 0.0;
            for (int j = lane; j < K; j += 64) {
                const double r = recip((dd[j] - dc) * (dd[j] + dc) - x), z = zz[j], tt = z * z * r;
                if (j <= i) {
                    psi += tt;
                    dpsi += tt * r;
                } else {
                    phi += tt;
                    dphi += tt * r;
                }
            }
            psi = wave_sum(psi);
            dpsi = wave_sum(dpsi);
            phi = wave_sum(phi);
            dphi = wave_sum(dphi);
            const double da = (di - dc) * (di + dc) - x, db = last ? 0.0 : (di1 - dc) * (di1 + dc) - x;
            if (root_step(x, lo, hi, psi, dpsi, phi, dphi, da, db, last)) break;
        }
        if (lane == 0) {
            sgo[g] = sigma_of(dc, x);
            w.x[g] = x;
            w.dc[g] = dc;
        }
        return;
    }
    const int gi = blockIdx.x - nroot, g = gi / nch;
    const Node nd = node_of(n, depth, g, q);
    if (q < 0) return;
    const int a = nd.a, m = nd.m, b = nd.b, s0i = g - a;
    const int c = a + (gi % nch) * 256 + threadIdx.x;
    if (c > b || c >= n || w.act[g] > 1) return;
    const bool null = b < n;
    const double c0 = w.cs[2 * q], s0 = w.cs[2 * q + 1];
    const double* __restrict__ U = w.UT[cur];
    const double* __restrict__ V = w.VT[cur];
    double* __restrict__ Uo = w.UT[cur ^ 1];
    double* __restrict__ Vo = w.VT[cur ^ 1];
    auto uat = [&](int r) {
        if (r == m) return c == m ? 1.0 : 0.0;
        return (r < m ? c < m : c > m) && c < b ? U[(long)r * n + c] : 0.0;
    };
    auto vat = [&](int r) {
        if (r == m) return c <= m ? c0 * V[(long)m * n + c] : (null ? s0 * V[(long)b * n + c] : 0.0);
        return (r < m ? c <= m : c > m) ? V[(long)r * n + c] : 0.0;
    };
    const int r = w.ord[g];
    double u = uat(r), v = vat(r);
    if (w.act[g] == 1) {
        const long at = (long)(a + w.dst[g]) * n + c;
        if (c < b) Uo[at] = u;
        Vo[at] = v;
        return;
    }
    if (s0i == 0 && null)
        Vo[(long)b * n + c] = c <= m ? -s0 * V[(long)m * n + c] : c0 * V[(long)b * n + c];
    for (int s = w.nxt[g]; s >= 0; s = w.nxt[a + s]) {
        const int rs = w.ord[a + s];
        const double cr = w.cr[a + s], sr = w.sr[a + s], us = uat(rs), vs = vat(rs);
        const long at = (long)(a + w.dst[a + s]) * n + c;
        if (w.act[a + s] == 3) {
            if (c < b) Uo[at] = us;
            Vo[at] = cr * vs - sr * v;
            v = cr * v + sr * vs;
        } else {
            if (c < b) Uo[at] = cr * u - sr * us;
            Vo[at] = cr * v - sr * vs;
            u = sr * u + cr * us;
            v = sr * v + cr * vs;
        }
    }
    const long at = (long)(a + w.dst[g]) * n + c;
    if (c < b) w.GU[at] = u;
    w.GV[at] = v;
}

// z of pole g recomputed from the roots, a wavefront each.
__global__ __launch_bounds__(256) void dc_zhat_kernel(DcWork w, int depth) {
    const int n = w.n, lane = threadIdx.x & 63, g = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= n) return;
    int q;
    const Node nd = node_of(n, depth, g, q);
    if (q < 0) return;
    const int K = w.K[q], i = g - nd.a;
    if (i >= K) return;
    const double* __restrict__ dd = w.dd + nd.a;
    const double* __restrict__ x = w.x + nd.a;
    const double* __restrict__ dc = w.dc + nd.a;
    const double di = dd[i];
    double p = 1.0;
    for (int k = lane; k < K; k += 64) {
        const double f = x[k] - (di - dc[k]) * (di + dc[k]);
        if (k == K - 1) p *= f;
        else {
            const double o = k < i ? dd[k] : dd[k + 1];
            p *= f * recip((o - di) * (o + di));
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) p *= __shfl_xor(p, o, 64);
    if (lane == 0) {
        const double z = sqrt(fabs(p));
        w.zh[g] = w.zz[g] < 0.0 ? -z : z;
    }
}

// Singular vectors of the merged matrix for root g, a wavefront each: row i
// of the node's K x K blocks in the children's (gathered) vector buffers.
__global__ __launch_bounds__(256) void dc_small_vectors_kernel(DcWork w, int depth, int cur) {
    const int n = w.n, lane = threadIdx.x & 63, g = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= n) return;
    int q;
    const Node nd = node_of(n, depth, g, q);
    if (q < 0) return;
    const int K = w.K[q], i = g - nd.a;
    if (i >= K) return;
    const double* __restrict__ dd = w.dd + nd.a;
    const double* __restrict__ zh = w.zh + nd.a;
    double* __restrict__ Us = w.UT[cur] + (long)g * n + nd.a;
    double* __restrict__ Vs = w.VT[cur] + (long)g * n + nd.a;
    if (K == 1) {
        if (lane == 0) {
            Us[0] = 1.0;
            Vs[0] = w.zz[g] < 0.0 ? -1.0 : 1.0;
        }
        return;
    }
    const double x = w.x[g], dc = w.dc[g];
    double nu = 0.0, nv = 0.0;
    for (int j = lane; j < K; j += 64) {
        const double d = dd[j], v = zh[j] * recip((d - dc) * (d + dc) - x), u = j == 0 ? -1.0 : d * v;
        nu += u * u;
        nv += v * v;
    }
    nu = 1.0 / sqrt(wave_sum(nu));
    nv = 1.0 / sqrt(wave_sum(nv));
    for (int j = lane; j < K; j += 64) {
        const double d = dd[j], v = zh[j] * recip((d - dc) * (d + dc) - x), u = j == 0 ? -1.0 : d * v;
        Us[j] = u * nu;
        Vs[j] = v * nv;
    }
}

// The node's vectors: (K x K) (K x N), blockIdx.z = 0 left, 1 right.
template <int BS>
__global__ __launch_bounds__(NTHREADS, 2) void dc_gemm_kernel(DcWork w, int depth, int cur) {
    constexpr int LDK = MfmaOp<double>::LDK;
    __shared__ __attribute__((aligned(16))) double As[2 * BS * LDK];
    __shared__ __attribute__((aligned(16))) double Bs[2 * BS * LDK];
    const int n = w.n, side = blockIdx.z;
    const Node nd = node_at(0, n, depth, blockIdx.y);
    const int K = w.K[blockIdx.y];
    const int cols = side ? min(nd.b, n - 1) - nd.a + 1 : nd.b - nd.a;
    const int nt = (cols + BS - 1) / BS, mt = (K + BS - 1) / BS;
    if ((int)blockIdx.x >= mt * nt) return;
    const long at = (long)nd.a * n + nd.a;
    const int tile = blockIdx.x;
    lds_tile<BS>((side ? w.VT[cur] : w.UT[cur]) + at, n, (side ? w.GV : w.GU) + at, n,
                 (side ? w.VT[cur ^ 1] : w.UT[cur ^ 1]) + at, n, K, cols, K, (tile / nt) * BS, (tile % nt) * BS, As, Bs);
}

int dc_depth(int n) {
    int depth = 0;
    for (int sz = n; sz > LEAF; sz /= 2) ++depth;
    return depth;
}

// Rank of every singular value by counting those before it (16 lanes a
// value, a pass over all n each): one launch for the order and the way to the
// host, where a copy, a sort there and a copy back took three and a wait.  The
// bits of the magnitudes order everything, NaN first (all values are NaN or none is).
__global__ __launch_bounds__(1024) void dc_sorted_kernel(const double* __restrict__ sg, int n,
                                                         const double* __restrict__ scale, int* __restrict__ perm,
                                                         HostPost post) {
    __shared__ double sorted[DC_POST];
    const int t = threadIdx.x, part = t & 15;
    const double f = *scale;
    auto key = [&](int i) { return (unsigned long long)__double_as_longlong(sg[i]) & 0x7fffffffffffffffull; };
    for (int i = blockIdx.x * 64 + (t >> 4); i < n; i += gridDim.x * 64) {
        const unsigned long long mine = key(i);
        int rank = 0;
        for (int j = part; j < n; j += 16) {
            const unsigned long long k = key(j);
            rank += k > mine || (k == mine && j < i);
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) rank += __shfl_xor(rank, o, 16);
        if (part == 0) {
            perm[rank] = i;
            if (post.flag) sorted[rank] = sg[i] * f;
            else post.data[rank] = sg[i] * f;
        }
    }
    if (!post.flag) return;
    __syncthreads();
    if (t < 64) {
        for (int i = t; i < n; i += 64) post.data[i] = sorted[i];
        if (t == 0) post_flag(post);
    }
}

}  // namespace

size_t dc_workspace(int n) {
    const size_t nn = n, nodes = (size_t)1 << dc_depth(n);
    return 6 * nn * nn + 14 * nn + 4 * nodes + 64 + (6 * nn + nodes) / 2 + 8;
}

DcWork dc_carve(double* ws, int n, const double* d, const double* e) {
    const size_t nn = (size_t)n * n, nodes = (size_t)1 << dc_depth(n);
    DcWork w{};
    w.n = n;
    w.d = d;
    w.e = e;
    double* p = ws;
    auto take = [&](size_t k) {
        double* r = p;
        p += k;
        return r;
    };
    for (int i = 0; i < 2; ++i) {
        w.UT[i] = take(nn);
        w.VT[i] = take(nn);
    }
    w.GU = take(nn);
    w.GV = take(nn);
    w.sg[0] = take(n);
    w.sg[1] = take(n);
    w.dd = take(n);
    w.zz = take(n);
    w.zh = take(n);
    w.x = take(n);
    w.dc = take(n);
    w.cr = take(n);
    w.sr = take(n);
    w.t0 = take(n);
    w.t1 = take(n);
    w.t2 = take(n);
    w.cs = take(2 * nodes);
    w.scale = take(1);
    w.inv = take(1);
    int* ip = reinterpret_cast<int*>(p);
    auto itake = [&](size_t k) {
        int* r = ip;
        ip += k;
        return r;
    };
    w.ord = itake(n);
    w.act = itake(n);
    w.dst = itake(n);
    w.nxt = itake(n);
    w.i0 = itake(n);
    w.i1 = itake(n);
    w.K = itake(nodes);
    return w;
}

void dc_sorted(const DcWork& w, int cur, int* perm, const HostPost& post, hipStream_t s) {
    const int blocks = w.n <= DC_POST ? 1 : (w.n + 63) / 64;
    hipLaunchKernelGGL(dc_sorted_kernel, dim3(blocks), dim3(1024), 0, s, w.sg[cur], w.n, w.scale, perm, post);
    HIP_CHECK(hipGetLastError());
}

int bidiagonal_svd(const DcWork& w, hipStream_t s, LaunchProbe* probe) {
    const int n = w.n, depth = dc_depth(n);
    bool timed = probe && probe->begin(PK_MERGE, s);
    hipLaunchKernelGGL(dc_leaf_kernel, dim3(1 << depth), dim3(LNT), 0, s, w, depth);
    if (timed) probe->end(PK_MERGE, s);
    int cur = 0;
    for (int dep = depth - 1; dep >= 0; --dep) {
        const int nodes = 1 << dep, most = (n >> dep) + 1, waves = (n + 3) / 4;
        const int nch = (most + 255) / 256;
        // (256 threads or 1024 for the order: no difference from 40 to 800 rows,
        // 110 and 110 us of merges at 100 rows, 448 and 433 at 800)
        timed = probe && probe->begin(PK_MERGE, s);
        if (most <= 256) hipLaunchKernelGGL((dc_prep_kernel<256>), dim3(nodes), dim3(256), 0, s, w, dep, cur);
        else hipLaunchKernelGGL((dc_prep_kernel<1024>), dim3(nodes), dim3(1024), 0, s, w, dep, cur);
        hipLaunchKernelGGL(dc_roots_kernel, dim3(waves + n * nch), dim3(256), 0, s, w, dep, cur, nch);
        hipLaunchKernelGGL(dc_zhat_kernel, dim3(waves), dim3(256), 0, s, w, dep);
        hipLaunchKernelGGL(dc_small_vectors_kernel, dim3(waves), dim3(256), 0, s, w, dep, cur);
        // tile by the node's rows; all merges of a block with one tile throughout (32,
        // 64, 128), us: 100 rows 107, 116, 135; 256 167, 178, 226; 512 246, 261, 362;
        // 1024 437, 450, 608; 2048 1312, 1268, 1450.  As taken: 512 306, 1024 551,
        // 2048 1400; the tiles want a better line than this one
        const int bs = most > 512 ? 128 : (most > 160 ? 64 : 32), tl = (most + bs - 1) / bs;
        const dim3 grid(tl * tl, nodes, 2);
        if (bs == 128) hipLaunchKernelGGL((dc_gemm_kernel<128>), grid, dim3(NTHREADS), 0, s, w, dep, cur);
        else if (bs == 64) hipLaunchKernelGGL((dc_gemm_kernel<64>), grid, dim3(NTHREADS), 0, s, w, dep, cur);
        else hipLaunchKernelGGL((dc_gemm_kernel<32>), grid, dim3(NTHREADS), 0, s, w, dep, cur);
        if (timed) probe->end(PK_MERGE, s);
        cur ^= 1;
    }
    HIP_CHECK(hipGetLastError());
    if (probe) {
        // without deflation the products of a level are 4 n^3 / 4^level flops
        double fl = 0.0;
        const double nd = n;
        for (int dep = 0; dep < depth; ++dep) fl += 4.0 * nd * nd * nd / (double)(1 << (2 * dep));
        probe->work(PK_MERGE, fl + 4.0 * nd * LEAF * LEAF, 8.0 * 6.0 * nd * nd);
    }
    return cur;
}

}  // namespace ite
