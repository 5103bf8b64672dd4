// Singular value decomposition of an upper bidiagonal matrix by divide and
// conquer (Gu and Eisenstat, "A divide-and-conquer algorithm for the
// bidiagonal SVD", SIAM J. Matrix Anal. Appl. 16, 1995).
//
// A node is a range [a, b) of rows with the columns [a, b] (without column n
// at the right end).  Its middle row m = a + (b - a) / 2 holds alpha = d_m in
// column m and beta = e_m in column m + 1; the rows before and after m are its
// children.  With the children's singular values and vectors, and their null
// vectors (a child has one column more than rows), the node's matrix becomes
// orthogonally equivalent to diag(0, d) with a first row z.  Entries with
// |z_j| below a few eps times the norm, and all but one of a group of equal
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
constexpr double DEFLATE = 8.0 * EPS;

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

__device__ inline double clean(double v) { return v == v ? v : 0.0; }

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
        eta = da + s / (1.0 + (psi - dpsi * da));
    } else {
        const double tt = dphi * db * db;
        const double cc = 1.0 + (psi - dpsi * da) + (phi - dphi * db);
        const double A = cc * (da + db) + s + tt, B = da * db * f;
        const double disc = sqrt(fmax(A * A - 4.0 * cc * B, 0.0));
        eta = A > 0.0 ? 2.0 * B / (A + disc) : (A - disc) / (2.0 * cc);
    }
    double xn = x + eta;
    if (!(xn > lo && xn < hi)) xn = 0.5 * (lo + hi);
    const bool done = xn == x || fabs(hi - lo) <= EPS * fabs(xn);
    x = xn;
    return done;
}
constexpr int ROOT_ITERS = 100;

// sigma from its pole and distance.
__device__ inline double sigma_of(double dc, double x) {
    const double s2 = dc * dc + x;
    return s2 > 0.0 ? dc + x / (dc + sqrt(s2)) : dc;
}

// ---------------------------------------------------------------------------
// Subtrees in LDS
// ---------------------------------------------------------------------------

// A level of a subtree in three steps: a wavefront a node sorts and deflates;
// then 32 lanes a row find the roots, recompute z and form the vectors (a pole
// each: a subtree has at most 32 rows, so the workgroup holds every row of
// the level whatever its nodes are); then a thread an entry of the products.
constexpr int LNT = LEAF * 32;
constexpr int LNW = LNT / 64;

struct LeafLDS {
    double U[2][LEAF][LEAF + 1], V[2][LEAF + 1][LEAF + 2];
    double Us[LEAF][LEAF + 1], Vs[LEAF][LEAF + 1];
    double sg[2][LEAF + 1], d[LEAF], e[LEAF];
    // a node's entries from its first row on: the order (scratch of its
    // wavefront), then poles, z and z recomputed
    double key[LEAF], sd[LEAF], sz[LEAF], cr[LEAF], sr[LEAF], dd[LEAF], zz[LEAF], zh[LEAF], x[LEAF], dc[LEAF];
    int srow[LEAF], prev[LEAF];
    int und[LEAF];                 // source row of the node's pole i: und[a + i]
    int kind[LEAF + 1], src[LEAF + 1], na[LEAF + 1], nb[LEAF + 1], nk[LEAF];
    double red[LNW];
};
enum { ROW_PRODUCT = 0, ROW_COPY = 1, ROW_NULL = 2 };

__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// Sort and deflation of one node of a subtree by one wavefront (local rows, at
// most 32).  `null`: column b exists.
__device__ __forceinline__ void leaf_deflate(LeafLDS& L, int cur, int a, int m, int b, bool null, int lane) {
    const int N = b - a;
    auto& U = L.U[cur];
    auto& V = L.V[cur];
    if (lane == 0 && null) {
        L.kind[b] = ROW_NULL;
        L.src[b] = b;
        L.na[b] = a;
        L.nb[b] = b;
    }
    if (N == 0) {
        if (null && lane <= LEAF) V[b][lane] = lane == b ? 1.0 : 0.0;
        return;
    }
    if (lane < N) {
        L.na[a + lane] = a;
        L.nb[a + lane] = b;
        L.kind[a + lane] = ROW_COPY;
        L.nk[a + lane] = 0;
    }
    const double alpha = L.d[m], beta = L.e[m];
    if (N == 1) {
        const double r = null ? hypot(alpha, beta) : fabs(alpha);
        double c = 1.0, s = 0.0;
        if (!null) c = alpha < 0.0 ? -1.0 : 1.0;
        else if (r > 0.0) {
            c = alpha / r;
            s = beta / r;
        }
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
    if (null) {
        r0 = hypot(x0, y0);
        if (r0 > 0.0) {
            c0 = x0 / r0;
            s0 = y0 / r0;
        }
    }
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
    double* key = L.key + a;
    double* sd = L.sd + a;
    double* sz = L.sz + a;
    int* srow = L.srow + a;
    if (lane < N) {
        U[m][a + lane] = a + lane == m ? 1.0 : 0.0;
        key[lane] = dv;
    }
    const double nrm = fmax(wave_max_nonneg(dv), fmax(fabs(clean(alpha)), fabs(clean(beta))));
    const double tol = DEFLATE * nrm;
    wave_fence();
    const int lm = m - a;
    if (lane < N) {
        int rank = lane == lm ? 0 : 1;
        for (int t = 0; t < N; ++t) {
            const double k = key[t];
            if (lane != lm && t != lm) rank += k < dv || (k == dv && t < lane);
        }
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
    const bool surv = lane > 0 && lane < N && fabs(zs) > tol;
    const bool tiny = surv && ds <= tol;
    const unsigned long long below = (1ull << lane) - 1;
    const unsigned long long ms = __ballot(surv && !tiny);
    int pv = -1;
    if (surv && !tiny) {
        const unsigned long long q = ms & below;
        pv = q ? 63 - __clzll(q) : -1;
        act = pv >= 0 && ds - sd[pv] <= tol ? 2 : 0;
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
                    const double zt = sz[t], tau = hypot(z, zt);
                    L.cr[a + t] = z / tau;
                    L.sr[a + t] = zt / tau;
                    z = tau;
                }
            } else if (m2) {
                const unsigned long long later = ms & ~below & ~(1ull << lane);
                for (unsigned long long q = later; q; q &= q - 1) {
                    const int t = __ffsll((long long)q) - 1;
                    if (!((m2 >> t) & 1)) break;
                    const double zt = sz[t], tau = hypot(z, zt);
                    L.cr[a + t] = zt / tau;
                    L.sr[a + t] = z / tau;
                    z = tau;
                    dl = sd[t];
                    last = srow[t];
                }
            }
            L.dd[a + slot] = dl;
            L.zz[a + slot] = z;
            L.und[a + slot] = last;
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

// Sums and products over the 32 lanes of a half wavefront, to all of them.
__device__ inline double half_sum(double v) {
    v += dpp_move<0xB1, 0xf>(v);
    v += dpp_move<0x4E, 0xf>(v);
    v += dpp_move<0x141, 0xf>(v);
    v += dpp_move<0x140, 0xf>(v);
    return v + __shfl_xor(v, 16, 32);
}
__device__ inline double half_product(double v) {
    v *= dpp_move<0xB1, 0xf>(v);
    v *= dpp_move<0x4E, 0xf>(v);
    v *= dpp_move<0x141, 0xf>(v);
    v *= dpp_move<0x140, 0xf>(v);
    return v * __shfl_xor(v, 16, 32);
}

// A power of two near the largest |d|, |e|.
__device__ inline double pow2_scale(double mx, bool inverse) {
    if (!(mx > 0.0) || !(mx < 1e300)) return 1.0;
    int ex;
    (void)frexp(mx, &ex);
    return ldexp(1.0, inverse ? -ex : ex);
}

__global__ __launch_bounds__(LNT) void dc_leaf_kernel(DcWork w, int depth) {
    __shared__ LeafLDS L;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, n = w.n;
    double mx = 0.0;
    for (int i = t; i < n; i += LNT) mx = fmax(mx, fmax(fabs(w.d[i]), i + 1 < n ? fabs(w.e[i]) : 0.0));
    mx = wave_max_nonneg(mx);
    if (lane == 0) L.red[wv] = mx;
    __syncthreads();
    mx = L.red[0];
    for (int q = 1; q < LNW; ++q) mx = fmax(mx, L.red[q]);
    const double inv = pow2_scale(mx, true);
    if (blockIdx.x == 0 && t == 0) {
        *w.scale = pow2_scale(mx, false);
        *w.inv = inv;
    }
    const Node root = node_at(0, n, depth, blockIdx.x);
    const int a0 = root.a, len = root.b - root.a;
    if (t < len) {
        L.d[t] = w.d[a0 + t] * inv;
        L.e[t] = a0 + t + 1 < n ? w.e[a0 + t] * inv : 0.0;
    }
    for (int x = t; x < 2 * LEAF * (LEAF + 1); x += LNT) (&L.U[0][0][0])[x] = 0.0;
    for (int x = t; x < 2 * (LEAF + 1) * (LEAF + 2); x += LNT) (&L.V[0][0][0])[x] = 0.0;
    __syncthreads();
    int top = 0;
    for (int sz = len; sz > 1; sz /= 2) ++top;
    int cur = 0;
    for (int lv = top; lv >= 0; --lv) {
        for (int q = wv; q < (1 << lv); q += LNW) {
            const Node nd = node_at(0, len, lv, q);
            leaf_deflate(L, cur, nd.a, nd.m, nd.b, a0 + nd.b < n, lane);
        }
        __syncthreads();
        // row r = t / 32 (a root, then a pole, then a root again), lane j a pole
        const int r = t >> 5, j = t & 31;
        const bool mine = r < len && L.kind[r] == ROW_PRODUCT;
        const int a = mine ? L.na[r] : 0, K = mine ? L.nk[r] : 0, i = r - a;
        const bool pole = mine && j < K;
        const double dj = pole ? L.dd[a + j] : 0.0, zj = pole ? L.zz[a + j] : 0.0, z2 = zj * zj;
        double x = 0.0, dc = 0.0;
        if (mine && K > 1) {
            const bool last = i == K - 1;
            const double di = L.dd[a + i], di1 = last ? 0.0 : L.dd[a + i + 1];
            double lo = 0.0, hi;
            dc = di;
            if (last) {
                hi = half_sum(z2) * (1.0 + 8.0 * EPS);
                x = 0.5 * hi;
            } else {
                const double mid = 0.5 * (di1 - di) * (di1 + di);
                const double f = 1.0 + half_sum(pole ? z2 * recip((dj - di) * (dj + di) - mid) : 0.0);
                hi = mid;
                x = mid;
                if (!(f >= 0.0)) {
                    dc = di1;
                    lo = -mid;
                    hi = 0.0;
                    x = -mid;
                }
            }
            const double del = (dj - dc) * (dj + dc);
            const double da0 = (di - dc) * (di + dc), db0 = last ? 0.0 : (di1 - dc) * (di1 + dc);
            for (int it = 0; it < ROOT_ITERS; ++it) {
                const double rc = pole ? recip(del - x) : 0.0, tt = z2 * rc, t2 = tt * rc;
                const double psi = half_sum(j <= i ? tt : 0.0), dpsi = half_sum(j <= i ? t2 : 0.0);
                const double phi = half_sum(j > i ? tt : 0.0), dphi = half_sum(j > i ? t2 : 0.0);
                if (root_step(x, lo, hi, psi, dpsi, phi, dphi, da0 - x, last ? 0.0 : db0 - x, last)) break;
            }
            if (j == 0) {
                L.sg[cur ^ 1][r] = sigma_of(dc, x);
                L.x[r] = x;
                L.dc[r] = dc;
            }
        } else if (mine && j == 0) {
            L.sg[cur ^ 1][r] = fabs(zj);
        }
        __syncthreads();
        if (mine && K > 1) {
            // z of pole i, lane j a root
            const double di = L.dd[a + i];
            double f = 1.0;
            if (pole) {
                f = L.x[a + j] - (di - L.dc[a + j]) * (di + L.dc[a + j]);
                if (j < K - 1) {
                    const double o = j < i ? dj : L.dd[a + j + 1];
                    f *= recip((o - di) * (o + di));
                }
            }
            f = sqrt(fabs(half_product(f)));
            if (j == 0) L.zh[r] = L.zz[r] < 0.0 ? -f : f;
        }
        __syncthreads();
        if (mine) {
            double u = 1.0, v = zj < 0.0 ? -1.0 : 1.0;
            if (K > 1) {
                v = pole ? L.zh[a + j] * recip((dj - dc) * (dj + dc) - x) : 0.0;
                u = j == 0 ? -1.0 : dj * v;
                u *= 1.0 / sqrt(half_sum(u * u));
                v *= 1.0 / sqrt(half_sum(v * v));
            }
            if (pole) {
                L.Us[r][j] = u;
                L.Vs[r][j] = v;
            }
        }
        __syncthreads();
        const int W = len + 1;
        const bool null = a0 + len < n;
        for (int e = t; e < W * W; e += LNT) {
            const int rr = e / W, c = e % W;
            if (rr == len && !null) continue;
            const int ra = L.na[rr], rb = L.nb[rr], kind = L.kind[rr];
            double u = 0.0, v = 0.0;
            if (c >= ra && c <= rb) {
                if (kind == ROW_PRODUCT) {
                    const int k = L.nk[rr];
                    for (int q = 0; q < k; ++q) {
                        const int g = L.und[ra + q];
                        u += L.Us[rr][q] * L.U[cur][g][c];
                        v += L.Vs[rr][q] * L.V[cur][g][c];
                    }
                } else {
                    const int g = L.src[rr];
                    if (kind == ROW_COPY) u = L.U[cur][g][c];
                    v = L.V[cur][g][c];
                }
            }
            if (rr < len && c < len) L.U[cur ^ 1][rr][c] = c < rb ? u : 0.0;
            L.V[cur ^ 1][rr][c] = v;
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
    if (null) {
        const double x0 = r0, y0 = beta * clean(VT[(long)b * n + m + 1]);
        r0 = hypot(x0, y0);
        if (r0 > 0.0) {
            c0 = x0 / r0;
            s0 = y0 / r0;
        }
    }
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
    const double tol = DEFLATE * fmax(mx, fmax(fabs(alpha), fabs(beta)));
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
        const bool surv = s > 0 && s < N && fabs(sz[s]) > tol, tiny = surv && sd[s] <= tol;
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
        act[s] = ci > 0 && sd[s] - sd[cl[ci - 1]] <= tol ? 2 : 0;
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
        const double zt = sz[s], tau = hypot(z, zt);
        w.cr[a + s] = (mid ? z : zt) / tau;
        w.sr[a + s] = (mid ? zt : z) / tau;
        z = tau;
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
                sgo[g] = fabs(zz[0]);
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
            const double mid = 0.5 * (di1 - di) * (di1 + di);
            double f = 0.0;
            for (int j = lane; j < K; j += 64) f += zz[j] * zz[j] * recip((dd[j] - di) * (dd[j] + di) - mid);
            f = 1.0 + wave_sum(f);
            hi = mid;
            x = mid;
            if (!(f >= 0.0)) {
                dc = di1;
                lo = -mid;
                hi = 0.0;
                x = -mid;
            }
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
    Params p;
    p.M = K;
    p.N = cols;
    p.K = K;
    p.alpha = 1.0;
    p.beta = 0.0;
    p.A = (side ? w.VT[cur] : w.UT[cur]) + at;
    p.B = (side ? w.GV : w.GU) + at;
    p.C = nullptr;
    p.D = (side ? w.VT[cur ^ 1] : w.UT[cur ^ 1]) + at;
    p.Df = nullptr;
    p.lda = p.ldb = p.ldc = p.ldd = n;
    p.sA = p.sB = p.sC = p.sD = 0;
    p.mt = mt;
    p.nt = nt;
    const int tile = blockIdx.x;
    gemm_tile<double, false, false, BS>(p, (tile / nt) * BS, (tile % nt) * BS, 0, As, Bs);
}

int dc_depth(int n) {
    int depth = 0;
    for (int sz = n; sz > LEAF; sz /= 2) ++depth;
    return depth;
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

int bidiagonal_svd(const DcWork& w, hipStream_t s, LaunchProbe* probe) {
    const int n = w.n, depth = dc_depth(n);
    bool timed = probe && probe->begin(PK_MERGE, s);
    hipLaunchKernelGGL(dc_leaf_kernel, dim3(1 << depth), dim3(LNT), 0, s, w, depth);
    if (timed) probe->end(PK_MERGE, s);
    int cur = 0;
    for (int dep = depth - 1; dep >= 0; --dep) {
        const int nodes = 1 << dep, most = (n >> dep) + 1, waves = (n + 3) / 4;
        const int nch = (most + 255) / 256;
        timed = probe && probe->begin(PK_MERGE, s);
        if (most <= 256) hipLaunchKernelGGL((dc_prep_kernel<256>), dim3(nodes), dim3(256), 0, s, w, dep, cur);
        else hipLaunchKernelGGL((dc_prep_kernel<1024>), dim3(nodes), dim3(1024), 0, s, w, dep, cur);
        hipLaunchKernelGGL(dc_roots_kernel, dim3(waves + n * nch), dim3(256), 0, s, w, dep, cur, nch);
        hipLaunchKernelGGL(dc_zhat_kernel, dim3(waves), dim3(256), 0, s, w, dep);
        hipLaunchKernelGGL(dc_small_vectors_kernel, dim3(waves), dim3(256), 0, s, w, dep, cur);
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
