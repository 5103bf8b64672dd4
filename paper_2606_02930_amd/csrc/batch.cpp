// Batched implicit steps for the serving path: several independent states
// sweep in lockstep, block slot by block slot, and the fixed-budget GMRES
// local solves of a slot run together -- one grouped launch per product
// stage (the uneven-bond-dimension H_eff products of all states), one
// batched launch per Krylov vector operation -- captured as a HIP graph per
// batch size, budget and precision (the last few kept per context) and
// replayed (the kernels read every shape and address from descriptors in
// device memory); a capture that a call on another thread invalidates is
// issued directly instead.  A
// product's tile and K parts depend on its shape alone, and every per-state
// reduction has the single-state partition and order, so a state's step does
// not depend on the batch it runs in.  FP32 refinement with a fixed number of corrections runs
// the same sequence with one cycle per correction: the residual product in
// FP64, the Arnoldi products with FP32 operands (grouped FP32 launches and the
// FP32 MPO stage), the Krylov basis and its reductions in FP64.
#include "engine.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>

namespace ite {

// ---------------------------------------------------------------------------
// Batched fixed-budget GMRES
// ---------------------------------------------------------------------------

namespace {

// The products of one batch: for product p (0: the residual's product with
// x, k + 1: the Arnoldi product with V_k) and each of the two GEMMs, the
// descriptors; counts[p][gemm] = {problems, tiles}; or, for blocks that take it
// in one launch, hd[p] and hc[p] = {problems, units}.
// With FP32 products (lo): for product p >= 1 and each GEMM one more
// descriptor set, counts_lo[p][gemm] = {problems, tiles}.
struct BatchLayout {
    size_t vec_off = 0, tot_off = 0, desc_off = 0, cnt_off = 0, hd_off = 0, hc_off = 0, dlo_off = 0, clo_off = 0,
           bytes = 0;
    int G = 0, np = 0;
    bool lo = false;
};

BatchLayout layout(int G, int np, bool lo) {
    BatchLayout l;
    l.G = G;
    l.np = np;
    l.lo = lo;
    auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
    l.vec_off = 0;
    l.tot_off = al(sizeof(BatchVec) * G);
    l.desc_off = al(l.tot_off + sizeof(int) * BT_N);
    l.cnt_off = al(l.desc_off + grouped_desc_bytes() * (size_t)np * 2 * G);
    l.hd_off = al(l.cnt_off + sizeof(int) * 2 * (size_t)np * 2);
    l.hc_off = al(l.hd_off + heff_desc_bytes() * (size_t)np * G);
    l.dlo_off = al(l.hc_off + sizeof(int) * 2 * (size_t)np);
    l.clo_off = al(l.dlo_off + (lo ? grouped_desc_bytes() * (size_t)np * 2 * G : 0));
    l.bytes = al(l.clo_off + sizeof(int) * 2 * (size_t)np * 2);
    return l;
}

// Kinds of launches a batch needs: the krylov_class bits, then the forms of H_eff.
constexpr unsigned BATCH_HEFF_SMALL = 16, BATCH_HEFF_LARGE = 32;

// The launch sequence of the batched solve on stream s; every argument is
// either fixed for the batch's size and budget or read from `dev`.
void issue(char* dev, const BatchLayout& l, unsigned classes, int mm, int max_cycles, hipStream_t s) {
    const auto* d = reinterpret_cast<const BatchVec*>(dev + l.vec_off);
    const int* tot = reinterpret_cast<const int*>(dev + l.tot_off);
    const int G = l.G;
    auto product = [&](int p) {
        if (l.lo && p > 0) {
            // FP32 operands: the vector rounded, L_lo x, the FP32 stage, x3 R_lo^T
            batch_vec(d, G, tot, 1, p - 1, s);
            for (int gm = 0; gm < 2; ++gm) {
                const int q = p * 2 + gm;
                const void* desc = dev + l.dlo_off + grouped_desc_bytes() * (size_t)q * G;
                const int* cnt = reinterpret_cast<const int*>(dev + l.clo_off) + 2 * q;
                gemm_grouped(desc, cnt, true, gm == 1, s);
                if (gm == 0) batch_stage_lo(d, G, tot, s);
            }
            return;
        }
        if (classes & BATCH_HEFF_SMALL)
            heff_grouped(dev + l.hd_off + heff_desc_bytes() * (size_t)p * G,
                         reinterpret_cast<const int*>(dev + l.hc_off) + 2 * p, s);
        for (int gm = 0; gm < 2 && (classes & BATCH_HEFF_LARGE); ++gm) {
            const int q = p * 2 + gm;
            const void* desc = dev + l.desc_off + grouped_desc_bytes() * (size_t)q * G;
            const int* cnt = reinterpret_cast<const int*>(dev + l.cnt_off) + 2 * q;
            gemm_grouped(desc, cnt, false, gm == 1, s);
            if (gm == 0) batch_stage(d, G, tot, s);
        }
    };
    for (int cyc = 0; cyc < max_cycles; ++cyc) {
        product(0);                              // V_0 = A x
        batch_start(d, G, tot, classes, mm, cyc == 0, s);
        for (int k = 0; k < mm; ++k) {
            product(k + 1);                      // w = A V_k
            batch_gram_schmidt(d, G, tot, classes, k, mm, s);
        }
        // mixed precision: the budget is the number of corrections, not a
        // GMRES budget, so its end sets no flag
        batch_hess(d, G, mm, true, !l.lo && cyc + 1 == max_cycles, s);
        batch_vec(d, G, tot, 0, mm, s);          // x += V y
    }
}

}  // namespace

void gmres_batch(ite_ctx* c, const std::vector<BatchItem>& items, int m, int max_cycles, bool lo) {
    const int G = (int)items.size();
    if (G == 0) return;
    const int mm = m;
    ITE_REQUIRE(mm >= 1 && mm <= 16, "gmres_batch: Krylov dimension must be in 1..16");
    // FP32 buffers of a problem, in doubles: rounded L and R, the rounded
    // vector, the FP32 intermediates
    auto lo_doubles = [&](const LocalOp& op, size_t n, size_t nxi) -> size_t {
        if (!lo) return 0;
        const size_t nl = (size_t)op.s.Dxl * op.s.w0 * op.s.Dyl, nr = (size_t)op.s.Dxr * op.s.w2 * op.s.Dyr;
        auto h = [](size_t nf) { return ((nf + 1) / 2 + 31) & ~size_t(31); };
        return h(nl) + h(nr) + h(n) + 2 * h(nxi);
    };
    // workspaces, carved from one slot
    auto al = [](size_t x) { return (x + 31) & ~size_t(31); };
    std::vector<size_t> off(G);
    size_t total = 0;
    for (int g = 0; g < G; ++g) {
        const LocalOp& op = items[g].op;
        const size_t n = op.n();
        ITE_REQUIRE((size_t)mm < n, "gmres_batch: Krylov dimension must be below the vector length");
        const int I = op.s.w0 * op.s.d1 * op.s.d2, O = op.s.d1 * op.s.d2 * op.s.w2;
        ITE_REQUIRE(I <= BATCH_STAGE_I, "gmres_batch: more than 128 MPO-stage inputs");
        const size_t nxi = (size_t)op.s.Dxl * std::max(I, O) * op.s.Dyr;
        off[g] = total;
        total += al((size_t)(mm + 1) * n) + al(n) + 2 * al(nxi) + al((size_t)reduce_blocks(n) * 64 + 64) +
                 al((size_t)mm * HESS_HC + 8) + al(64) + lo_doubles(op, n, nxi);
    }
    double* ws = slot_t<double>(c, SL_BATCH, total);
    const int np = mm + 1;
    const BatchLayout lay = layout(G, np, lo);
    char* dev = static_cast<char*>(slot(c, SL_BDESC, lay.bytes));
    std::vector<char>& host = c->batch_host;
    host.assign(lay.bytes, 0);
    auto* hv = reinterpret_cast<BatchVec*>(host.data() + lay.vec_off);
    int* htot = reinterpret_cast<int*>(host.data() + lay.tot_off);
    int* hcnt = reinterpret_cast<int*>(host.data() + lay.cnt_off);
    std::vector<double*> X1(G), X3(G);
    std::vector<float*> Llo(G), Rlo(G), X1lo(G), X3lo(G);
    int red = 0, ew = 0, stg = 0, stg_lo = 0;
    std::vector<char> small(G);
    unsigned classes = 0;
    for (int g = 0; g < G; ++g) {
        const LocalOp& op = items[g].op;
        const size_t n = op.n();
        const int I = op.s.w0 * op.s.d1 * op.s.d2, O = op.s.d1 * op.s.d2 * op.s.w2;
        const size_t nxi = (size_t)op.s.Dxl * std::max(I, O) * op.s.Dyr;
        double* q = ws + off[g];
        BatchVec& v = hv[g];
        v = BatchVec{};   // the stage's default strides (the buffer itself is zeroed bytes)
        v.n = (long)n;
        v.nb = reduce_blocks(n);
        classes |= 1u << krylov_class(n);
        v.V = q;
        q += al((size_t)(mm + 1) * n);
        v.w = q;
        q += al(n);
        X1[g] = q;
        q += al(nxi);
        X3[g] = q;
        q += al(nxi);
        v.part = q;
        q += al((size_t)v.nb * 64 + 64);
        v.hd = q;
        q += al((size_t)mm * HESS_HC + 8);
        v.y = q;
        q += al(64);
        if (lo) {
            auto take = [&](size_t nf) {
                float* f = reinterpret_cast<float*>(q);
                q += ((nf + 1) / 2 + 31) & ~size_t(31);
                return f;
            };
            const size_t nl = (size_t)op.s.Dxl * op.s.w0 * op.s.Dyl, nr = (size_t)op.s.Dxr * op.s.w2 * op.s.Dyr;
            Llo[g] = take(nl);
            Rlo[g] = take(nr);
            v.tlo = take(n);
            X1lo[g] = take(nxi);
            X3lo[g] = take(nxi);
            // the environments rounded once per solve, ordered before it
            convert_f32(op.L, Llo[g], nl, c->stream);
            convert_f32(op.R, Rlo[g], nr, c->stream);
        }
        v.x = items[g].x;
        v.b = items[g].b;
        v.stats = items[g].stats;
        Stage& st = v.st;
        st.G = op.s.Dxl;
        st.C = op.s.Dyr;
        st.in = X1[g];
        st.in_gs = (long)I * op.s.Dyr;
        st.in_s1 = op.s.Dyr;
        st.out = X3[g];
        st.out_gs = (long)O * op.s.Dyr;
        st.out_s1 = op.s.Dyr;
        st.I = op.ww->I;
        st.O = op.ww->O;
        st.rowptr = op.ww->rowptr;
        st.col = op.ww->col;
        st.val = op.ww->val;
        st.nnz = op.ww->nnz;
        st.csr_lds = st.nnz >= 0 && (size_t)st.nnz * 12 + (size_t)(st.O + 1) * 4 <= BATCH_STAGE_CSR;
        if (lo) {
            Stage& sl = v.st_lo;
            sl = st;
            sl.in = nullptr;
            sl.in_f32 = X1lo[g];
            sl.out = nullptr;
            sl.out_prec = 1;
            sl.out_lo = X3lo[g];
        }
        v.red_start = red;
        v.ew_start = ew;
        v.stage_start = stg;
        v.stage_lo_start = stg_lo;
        red += v.nb;
        ew += (int)((n + BATCH_EW - 1) / BATCH_EW);
        const int units = op.s.Dxl * ((op.s.Dyr + (1 << BATCH_STAGE_LC) - 1) >> BATCH_STAGE_LC);
        stg_lo += units;
        small[g] = heff_small_ok(heff_small_of(op.s, op.L, *op.ww, op.R, nullptr, 0.0, 0.0, nullptr, nullptr));
        if (!small[g]) stg += units;
        classes |= small[g] ? BATCH_HEFF_SMALL : BATCH_HEFF_LARGE;
    }
    htot[BT_RED] = red;
    htot[BT_EW] = ew;
    htot[BT_STAGE] = stg;
    htot[BT_STAGE_LO] = stg_lo;
    // grouped products: theta = x (p = 0) or V_(p-1), into V_0 or w
    std::vector<Gemm> g1(G), g2(G);
    for (int g = 0; g < G; ++g) {
        const LocalOp& op = items[g].op;
        const HeffShape& s = op.s;
        Gemm& a = g1[g];
        a.M = s.Dxl * s.w0;
        a.N = s.d1 * s.d2 * s.Dyr;
        a.K = s.Dyl;
        a.alpha = 1.0;
        a.beta = 0.0;
        a.A = op.L;
        a.lda = s.Dyl;
        a.ldb = (long)s.d1 * s.d2 * s.Dyr;
        a.D = X1[g];
        a.ldd = a.ldb;
        Gemm& b = g2[g];
        b.M = s.Dxl * s.d1 * s.d2;
        b.N = s.Dxr;
        b.K = s.w2 * s.Dyr;
        b.tB = true;
        b.alpha = op.beta;
        b.beta = op.alpha;
        b.A = X3[g];
        b.lda = (long)s.w2 * s.Dyr;
        b.B = op.R;
        b.ldb = b.lda;
        b.ldc = s.Dxr;
        b.ldd = s.Dxr;
    }
    int* hhc = reinterpret_cast<int*>(host.data() + lay.hc_off);
    for (int p = 0; p < np; ++p) {
        auto theta = [&](int g) -> const double* {
            return p == 0 ? items[g].x : hv[g].V + (size_t)(p - 1) * hv[g].n;
        };
        auto out = [&](int g) { return p == 0 ? hv[g].V : hv[g].w; };
        for (int gm = 0; gm < 2; ++gm) {
            const int q = p * 2 + gm;
            char* desc = host.data() + lay.desc_off + grouped_desc_bytes() * (size_t)q * G;
            int cnt = 0, tiles = 0;
            for (int g = 0; g < G; ++g) {
                if (small[g]) continue;
                Gemm e = gm == 0 ? g1[g] : g2[g];
                if (gm == 0) e.B = theta(g);
                else {
                    e.C = theta(g);
                    e.D = out(g);
                }
                tiles += grouped_desc_fill(e, false, tiles, desc + grouped_desc_bytes() * cnt++);
            }
            hcnt[2 * q] = cnt;
            hcnt[2 * q + 1] = tiles;
        }
        char* desc = host.data() + lay.hd_off + heff_desc_bytes() * (size_t)p * G;
        int cnt = 0, units = 0;
        for (int g = 0; g < G; ++g) {
            if (!small[g]) continue;
            const LocalOp& op = items[g].op;
            const HeffSmall h = heff_small_of(op.s, op.L, *op.ww, op.R, theta(g), op.beta, op.alpha, theta(g), out(g));
            units += heff_desc_fill(h, units, desc + heff_desc_bytes() * cnt++);
        }
        hhc[2 * p] = cnt;
        hhc[2 * p + 1] = units;
    }
    if (lo) {
        // FP32 products p >= 1: L_lo tlo -> X1lo (FP32), X3lo R_lo^T + (1 - h s) V_(p-1) -> w
        int* hclo = reinterpret_cast<int*>(host.data() + lay.clo_off);
        for (int p = 1; p < np; ++p)
            for (int gm = 0; gm < 2; ++gm) {
                const int q = p * 2 + gm;
                char* desc = host.data() + lay.dlo_off + grouped_desc_bytes() * (size_t)q * G;
                int tiles = 0;
                for (int g = 0; g < G; ++g) {
                    Gemm e = gm == 0 ? g1[g] : g2[g];
                    if (gm == 0) {
                        e.A = Llo[g];
                        e.B = hv[g].tlo;
                        e.D = nullptr;
                        e.Df = X1lo[g];
                    } else {
                        e.A = X3lo[g];
                        e.B = Rlo[g];
                        e.C = hv[g].V + (size_t)(p - 1) * hv[g].n;
                        e.D = hv[g].w;
                    }
                    tiles += grouped_desc_fill(e, true, tiles, desc + grouped_desc_bytes() * g);
                }
                hclo[2 * q] = G;
                hclo[2 * q + 1] = tiles;
            }
    }
    // upload (ordered before the solve on the context's stream), then run the
    // sequence on the private stream, captured once per batch size, budget,
    // precision and kinds of vectors
    HIP_CHECK(hipMemcpyAsync(dev, host.data(), lay.bytes, hipMemcpyHostToDevice, c->stream));
    c->batch_solves++;
    if (!c->use_graphs) {
        issue(dev, lay, classes, mm, max_cycles, c->stream);
        return;
    }
    if (!c->side) {
        HIP_CHECK(hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking));
        HIP_CHECK(hipEventCreateWithFlags(&c->ev_in, hipEventDisableTiming));
        HIP_CHECK(hipEventCreateWithFlags(&c->ev_out, hipEventDisableTiming));
    }
    const long long key[5] = {G, mm + (lo ? 1000 : 0) + 2000 * (int)classes, max_cycles, (long long)(uintptr_t)dev, (long long)lay.bytes};
    auto& cache = c->bgraphs;
    auto hit = std::find_if(cache.begin(), cache.end(),
                            [&](const ite_ctx::BatchGraph& e) { return std::memcmp(key, e.key, sizeof(key)) == 0; });
    hipGraphExec_t exec = nullptr;
    if (hit != cache.end()) {
        ite_ctx::BatchGraph e = *hit;   // most recently used to the back
        cache.erase(hit);
        cache.push_back(e);
        exec = e.exec;
    } else {
        if ((int)cache.size() >= BGRAPH_CACHE) {
            HIP_CHECK(hipStreamSynchronize(c->side));
            HIP_CHECK(hipGraphExecDestroy(cache.front().exec));
            cache.erase(cache.begin());
        }
        hipGraph_t graph = nullptr;
        HIP_CHECK(hipStreamBeginCapture(c->side, hipStreamCaptureModeThreadLocal));
        bool ok = true;
        try {
            issue(dev, lay, classes, mm, max_cycles, c->side);
        } catch (const Error&) {
            ok = false;
        }
        if (hipStreamEndCapture(c->side, &graph) != hipSuccess || !graph) ok = false;
        if (ok && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) {
            ok = false;
            exec = nullptr;
        }
        if (graph) (void)hipGraphDestroy(graph);
        if (!ok) {
            // a call on another thread that a capture does not allow can end
            // or spoil it; nothing captured ran, so the same sequence is
            // issued directly (where a genuine launch error surfaces)
            (void)hipGetLastError();
            c->graph_fallbacks++;
            issue(dev, lay, classes, mm, max_cycles, c->stream);
            return;
        }
        ite_ctx::BatchGraph ent;
        std::memcpy(ent.key, key, sizeof(key));
        ent.exec = exec;
        cache.push_back(ent);
        c->graph_captures++;
    }
    HIP_CHECK(hipEventRecord(c->ev_in, c->stream));
    HIP_CHECK(hipStreamWaitEvent(c->side, c->ev_in, 0));
    HIP_CHECK(hipGraphLaunch(exec, c->side));
    HIP_CHECK(hipEventRecord(c->ev_out, c->side));
    HIP_CHECK(hipStreamWaitEvent(c->stream, c->ev_out, 0));
    c->graph_replays++;
}

}  // namespace ite
