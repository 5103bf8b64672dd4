"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values; `kind` says which entry point it goes through:

* ``evolve`` -- a product state evolved over a whole small grid at complete
  bonds with tolerance-driven local solves (the L = 10 chain of the workloads:
  short vectors, where launches and host round trips set the time);
* ``step``   -- one trapezoid step of a state that a program holds as a
  checkpoint (load, step with the paper's budget and cutoff, export): chains
  of the Heisenberg model (d = 2) and the Anderson impurity model (d = 4) at
  the bond dimensions of the serving stream and of the adaptive runs;
* ``batch``  -- one step of several uneven chains at once, as the server
  advances its active requests;
* ``solve``  -- one local GMRES solve of a block in FP64 (the paper's fixed
  budget) or with FP32 / BF16 products refined to an FP64 residual;
* ``split``  -- the truncated SVD of one two-site block, both directions;
* ``sample`` -- product-basis samples of a state (the METTS collapse).

States are random right-orthonormal MPS whose Schmidt values fall like
exp(-a ln^2 k), the shape of an entanglement spectrum, and reach the square
root of the cutoff near the bond cap, so that the caps are in use.  Results that carry a
gauge (the bond bases of an MPS, the signs of singular vectors) are returned as
what they represent: the state's amplitudes, the truncated block and the
overlaps of its basis vectors.
"""
import math
import weakref

import numpy as np
import torch

import paper_2606_02930_amd as ite
from paper_2606_02930_amd import hamiltonians

_SPLIT_RATE = 0.35      # a of exp(-a ln^2 k) for a block's singular values

_PREC = {"fp64": ite.PREC_FP64, "fp32": ite.PREC_FP32_IR, "bf16": ite.PREC_BF16_IR}


def listed():
    return [
        # the smallest whole evolution: L = 10 at complete bonds, backward Euler
        # solved to 1e-12 (the workload that is checked against exact
        # diagonalisation)
        {"name": "evolve_L10_chi32", "kind": "evolve", "L": 10, "chi": 32, "tau0": 0.1, "tau1": 1.0, "ratio": 1.5},
        # a serving-size step (the scaled-down request stream: L in 12..24, chi in 16..32)
        {"name": "step_L16_chi32", "kind": "step", "model": "heisenberg", "L": 16, "chi": 32, "h": 0.05},
        # the adaptive-bond step of the paper's Heisenberg run (bonds of about 120)
        {"name": "step_L20_chi120", "kind": "step", "model": "heisenberg", "L": 20, "chi": 120, "h": 0.05},
        # the bond cap of the L = 64 workload
        {"name": "step_L22_chi256", "kind": "step", "model": "heisenberg", "L": 22, "chi": 256, "h": 0.05},
        # the impurity model (d = 4, MPO bond 6) at the bonds where its runs settle
        {"name": "step_aim8_chi64", "kind": "step", "model": "aim", "L": 8, "chi": 64, "h": 0.05},
        # a worker's active requests advanced together
        {"name": "batch_6_L12_16", "kind": "batch", "n": 6, "L": 14, "chi": 32, "h": 0.05},
        # the local solve of the headline block (bond 1024, 86.7 GFLOP per product)
        {"name": "solve_fp64_1024", "kind": "solve", "prec": "fp64", "Dl": 1024, "Dr": 1024, "d": 2, "w": 5},
        # mixed precision on ragged bonds, refined to an FP64 residual of 1e-12
        {"name": "solve_fp32_383x401", "kind": "solve", "prec": "fp32", "Dl": 383, "Dr": 401, "d": 2, "w": 5},
        # the impurity model's block with BF16 products, refined likewise
        {"name": "solve_bf16_256_d4", "kind": "solve", "prec": "bf16", "Dl": 256, "Dr": 256, "d": 4, "w": 6},
        # the bond truncation of the headline block (2048 x 2048, 1024 kept)
        {"name": "split_2048", "kind": "split", "Dl": 1024, "d1": 2, "d2": 2, "Dr": 1024, "chi": 1024, "cutoff": 0.0,
         "spectrum": "graded", "dir": 0},
        # the truncation of the adaptive runs (about 220 x 220), right-to-left, odd bonds
        {"name": "split_218x226", "kind": "split", "Dl": 109, "d1": 2, "d2": 2, "Dr": 113, "chi": 128,
         "cutoff": 1e-10, "spectrum": "graded", "dir": 1},
        # the collapse of a METTS chain: 1024 samples at once
        {"name": "sample_L64_chi256", "kind": "sample", "L": 64, "chi": 256, "n": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "split", "split", "split", "solve", "solve", "batch", "sample"])
    if kind == "step":
        if rng.random() < 0.7:
            return {"kind": "step", "model": "heisenberg", "L": rng.randint(8, 22), "chi": _log_int(rng, 8, 200),
                    "h": round(rng.uniform(0.01, 0.1), 3)}
        return {"kind": "step", "model": "aim", "L": rng.randint(5, 8), "chi": _log_int(rng, 8, 64),
                "h": round(rng.uniform(0.01, 0.1), 3)}
    if kind == "batch":
        return {"kind": "batch", "n": rng.randint(2, 8), "L": rng.randint(8, 16), "chi": _log_int(rng, 8, 48),
                "h": round(rng.uniform(0.01, 0.1), 3)}
    if kind == "solve":
        d, w = rng.choice([(2, 5), (2, 5), (4, 6)])
        top = 1000 if d == 2 else 300
        return {"kind": "solve", "prec": rng.choice(["fp64", "fp64", "fp32", "bf16"]), "Dl": _log_int(rng, 8, top),
                "Dr": _log_int(rng, 8, top), "d": d, "w": w}
    if kind == "split":
        d = rng.choice([2, 2, 4])
        top = 1600 // d
        dl, dr = _log_int(rng, 4, top), _log_int(rng, 4, top)
        return {"kind": "split", "Dl": dl, "d1": d, "d2": d, "Dr": dr, "chi": max(1, d * min(dl, dr) * 2 // 3),
                "cutoff": rng.choice([0.0, 1e-10]), "spectrum": rng.choice(["graded", "graded", "flat"]),
                "dir": rng.randint(0, 1)}
    return {"kind": "sample", "L": rng.randint(16, 80), "chi": _log_int(rng, 16, 240), "n": _log_int(rng, 16, 1000)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

_context = []


def _ctx():
    """The one context a program keeps per host thread."""
    if not _context:
        _context.append(ite.ite_ctx_create(0))
    return _context[0]


class _State:
    """What a program holds between calls; releases its library handles."""

    def __init__(self, **kw):
        self.__dict__.update(kw)
        for h in kw.get("mpos", []):
            weakref.finalize(self, ite.ite_mpo_destroy, h)
        for h in kw.get("held", []):
            weakref.finalize(self, ite.ite_mps_destroy, h)


def _model(case, L):
    if case.get("model", "heisenberg") == "heisenberg":
        return hamiltonians.heisenberg(L)
    eps = -1.0 + 2.0 * (np.arange(L - 1) + 0.5) / (L - 1)
    return hamiltonians.anderson_star(4.0, -2.0, eps, np.full(L - 1, 0.25))


def _graded_mps(rng, L, d, chi):
    """Right-orthonormal MPS, norm 1 on site 1, with decaying Schmidt values."""
    dims = [int(min(chi, float(d) ** i, float(d) ** (L - i))) for i in range(L + 1)]
    # 3.4: the exponent at which the Schmidt values of such states reach about 1e-5 at k = chi
    rate = 0.5 * 3.4 / math.log(max(chi, 4)) ** 2
    lam = [np.exp(-rate * np.log(np.arange(1, D + 1)) ** 2) for D in dims]
    out = [None] * L
    carry = np.ones((1, 1))
    for i in range(L - 1, -1, -1):
        g = rng.standard_normal((dims[i], d, dims[i + 1])) * lam[i][:, None, None] * lam[i + 1][None, None, :]
        a = np.tensordot(g, carry, axes=([2], [0])).reshape(dims[i], -1)
        if i == 0:
            out[0] = (a / np.linalg.norm(a)).reshape(1, d, -1)
            break
        q, r = np.linalg.qr(a.T)
        out[i] = np.ascontiguousarray(q.T).reshape(dims[i], d, -1)
        carry = r.T / np.linalg.norm(r)
    return out


def _spinors(rng, L, d):
    v = rng.standard_normal((L, d))
    return [x / np.linalg.norm(x) for x in v]


def _boundary(g, D, w, flip):
    """A boundary environment [D][w][D] of a nearest-neighbour-like Hamiltonian:
    the identity at one end of the MPO index, the accumulated Hamiltonian
    (symmetric, spectrum within about [-1, 1]) at the other, pairs of mutually
    transposed operators and symmetric ones between."""
    def rand():
        return torch.randn((D, D), dtype=torch.float64, device="cuda", generator=g) / (2.0 * math.sqrt(2.0 * D))
    ops = []
    first, last = (w - 1, 0) if flip else (0, w - 1)
    pair = None
    for k in range(w):
        if k == first:
            ops.append(torch.eye(D, dtype=torch.float64, device="cuda"))
        elif k == last:
            a = rand()
            ops.append(a + a.T)
        elif pair is not None:
            ops.append(pair.T)
            pair = None
        elif k + 1 < w and k + 1 not in (first, last):
            pair = rand()
            ops.append(pair)
        else:
            a = rand()
            ops.append(0.5 * (a + a.T))
    return torch.stack(ops, dim=1).contiguous()


def _solve_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    W = _model({"model": "heisenberg" if case["d"] == 2 else "aim"}, 5)
    L = _boundary(g, case["Dl"], case["w"], False)
    R = _boundary(g, case["Dr"], case["w"], True)
    b = torch.randn((case["Dl"], case["d"], case["d"], case["Dr"]), dtype=torch.float64, device="cuda", generator=g)
    b /= b.norm()
    return L, R, W[2], W[3], b


def _theta(case, seed):
    m, n = case["Dl"] * case["d1"], case["d2"] * case["Dr"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["spectrum"] == "flat":
        t = torch.randn((m, n), dtype=torch.float64, device="cuda", generator=g)
    else:
        r = min(m, n)
        s = torch.exp(-_SPLIT_RATE * torch.log(torch.arange(1, r + 1, dtype=torch.float64, device="cuda")) ** 2)
        t = (torch.randn((m, r), dtype=torch.float64, device="cuda", generator=g) * s) @ \
            torch.randn((r, n), dtype=torch.float64, device="cuda", generator=g)
    return (t / t.norm()).reshape(case["Dl"], case["d1"], case["d2"], case["Dr"]).contiguous()


def _step_opts(case):
    return ite.ite_default_opts(chi_max=case["chi"], cutoff=1e-10)


def _batch_sizes(case):
    """The chains of a batch: lengths and bond caps around the case's."""
    return [(max(4, case["L"] - 2 + (2 * j) % 5), max(4, case["chi"] - 3 * j)) for j in range(case["n"])]


def prepare(case, seed):
    ctx = _ctx()
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "evolve":
        o = ite.ite_default_opts(scheme=ite.SCHEME_BE, shift_mode=ite.SHIFT_TRACK, chi_max=case["chi"], cutoff=0.0,
                                 max_cycles=100, tol_loc=1e-12)
        return _State(case=case, spinors=_spinors(rng, case["L"], 2), opts=o,
                      mpos=[ite.ite_mpo_load(ctx, _model(case, case["L"]))])
    if kind == "step":
        d = 2 if case["model"] == "heisenberg" else 4
        return _State(case=case, d=d, tensors=_graded_mps(rng, case["L"], d, case["chi"]), opts=_step_opts(case),
                      mpos=[ite.ite_mpo_load(ctx, _model(case, case["L"]))])
    if kind == "batch":
        sizes = _batch_sizes(case)
        return _State(case=case, sizes=sizes, tensors=[_graded_mps(rng, L, 2, chi) for L, chi in sizes],
                      opts=[_step_opts({"chi": chi}) for _, chi in sizes],
                      mpos=[ite.ite_mpo_load(ctx, _model(case, L)) for L, _ in sizes])
    if kind == "solve":
        L, R, W1, W2, b = _solve_inputs(case, seed)
        return _State(case=case, L=L, R=R, W1=W1, W2=W2, b=b, x=torch.empty_like(b))
    if kind == "split":
        th = _theta(case, seed)
        r = min(case["Dl"] * case["d1"], case["d2"] * case["Dr"], case["chi"])
        return _State(case=case, theta=th, A1=torch.zeros(case["Dl"] * case["d1"] * r, dtype=torch.float64, device="cuda"),
                      A2=torch.zeros(r * case["d2"] * case["Dr"], dtype=torch.float64, device="cuda"))
    psi = ite.ite_mps_load(ctx, _graded_mps(rng, case["L"], 2, case["chi"]), case["chi"])
    return _State(case=case, held=[psi], uniforms=rng.random((case["L"], case["n"])))


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _amplitudes(tensors):
    """Every amplitude of a short chain's state, on the GPU."""
    half = len(tensors) // 2
    parts = []
    for group in (tensors[:half], tensors[half:]):
        v = torch.from_numpy(group[0]).cuda()
        for a in group[1:]:
            v = v.reshape(-1, v.shape[-1]) @ torch.from_numpy(a).cuda().reshape(a.shape[0], -1)
            v = v.reshape(-1, a.shape[2])
        parts.append(v)
    left = parts[0].reshape(-1, tensors[half].shape[0])
    return (left @ parts[1].reshape(tensors[half].shape[0], -1)).reshape(-1)


def _numbers(rep):
    return {k: rep[k] for k in ("tau", "energy", "norm_before", "shift")}


def run(state):
    ctx, case = _ctx(), state.case
    kind = case["kind"]
    if kind == "evolve":
        psi = ite.ite_mps_create(ctx, state.spinors, case["chi"], pad_full=True)
        reps = ite.ite_evolve_loggrid(ctx, psi, state.mpos[0], case["tau0"], case["tau1"], case["ratio"], state.opts)
        out = ite.ite_mps_export(ctx, psi, [2] * case["L"])
        ite.ite_mps_destroy(psi)
        return {"psi": _amplitudes(out), "energy": np.array([r["energy"] for r in reps])}
    if kind == "step":
        psi = ite.ite_mps_load(ctx, state.tensors, case["chi"])
        rep = ite.ite_imag_step(ctx, psi, state.mpos[0], case["h"], state.opts)
        out = ite.ite_mps_export(ctx, psi, [state.d] * case["L"])
        ite.ite_mps_destroy(psi)
        return {"psi": _amplitudes(out), **_numbers(rep)}
    if kind == "batch":
        psis = [ite.ite_mps_load(ctx, t, chi) for t, (_, chi) in zip(state.tensors, state.sizes)]
        reps, _ = ite.ite_step_batch(ctx, psis, state.mpos, [case["h"]] * case["n"], state.opts)
        outs = [ite.ite_mps_export(ctx, p, [2] * L) for p, (L, _) in zip(psis, state.sizes)]
        for p in psis:
            ite.ite_mps_destroy(p)
        return [{"psi": _amplitudes(o), **_numbers(r)} for o, r in zip(outs, reps)]
    if kind == "solve":
        lo = case["prec"] != "fp64"
        _, res = ite.ite_debug_local_solve(ctx, state.L, state.W1, state.W2, state.R, 1.1, 0.1, state.b, state.b,
                                           state.x, krylov_dim=10, max_cycles=1, precision=_PREC[case["prec"]],
                                           max_refine=12 if lo else 1, tol_refine=1e-12 if lo else 0.0)
        return {"x": state.x}
    if kind == "split":
        k, sigma, disc = ite.ite_debug_svd_split(ctx, case["dir"], state.theta, case["chi"], case["cutoff"], 1e-13,
                                                 state.A1, state.A2)
        m, n = case["Dl"] * case["d1"], case["d2"] * case["Dr"]
        a1, a2 = state.A1[: m * k].view(m, k), state.A2[: k * n].view(k, n)
        basis = a1.T @ a1 if case["dir"] == 0 else a2 @ a2.T
        return {"theta": a1 @ a2, "basis": basis, "sigma": sigma, "k": k, "disc": disc}
    return {"configs": ite.ite_mps_sample(ctx, state.held[0], state.uniforms)}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _heisenberg_dense(L):
    sz = torch.diag(torch.tensor([0.5, -0.5], dtype=torch.float64))
    sp = torch.zeros((2, 2), dtype=torch.float64)
    sp[0, 1] = 1.0
    sm = sp.T.contiguous()
    H = torch.zeros((2 ** L, 2 ** L), dtype=torch.float64)
    for j in range(L - 1):
        bond = torch.kron(sz, sz) + 0.5 * (torch.kron(sp, sm) + torch.kron(sm, sp))
        H += torch.kron(torch.kron(torch.eye(2 ** j, dtype=torch.float64), bond),
                        torch.eye(2 ** (L - 2 - j), dtype=torch.float64))
    return H


def _exact_evolve(case, seed):
    L = case["L"]
    psi = torch.ones(1, dtype=torch.float64)
    for s in _spinors(np.random.default_rng(seed), L, 2):
        psi = torch.kron(psi, torch.from_numpy(s))
    H = _heisenberg_dense(L)
    eye = torch.eye(2 ** L, dtype=torch.float64)
    taus, t = [0.0], case["tau0"]
    while t < case["tau1"] * (1 - 1e-12):
        taus.append(t)
        t *= case["ratio"]
    taus.append(case["tau1"])
    energies = []
    E = float(psi @ (H @ psi))
    for a, b in zip(taus, taus[1:]):
        psi = torch.linalg.solve(eye + (b - a) * (H - E * eye), psi)
        psi = psi / psi.norm()
        E = float(psi @ (H @ psi))
        energies.append(E)
    return {"psi": psi, "energy": np.array(energies)}


def _exact_solve(case, seed):
    L, R, W1, W2, b = _solve_inputs(case, seed)
    Dl, Dr, d = case["Dl"], case["Dr"], case["d"]
    w0, w2 = W1.shape[0], W2.shape[1]
    pair = np.tensordot(W1, W2, axes=([1], [0]))                       # w p s u q t
    M = torch.from_numpy(np.ascontiguousarray(pair.transpose(1, 4, 3, 0, 2, 5))).cuda().reshape(d * d * w2, w0 * d * d)
    R2 = R.permute(1, 2, 0).reshape(w2 * Dr, Dr).contiguous()          # (u c) -> c'

    def apply(v):
        x = (L.reshape(Dl * w0, Dl) @ v.reshape(Dl, -1)).reshape(Dl, w0 * d * d, Dr)
        x = (M @ x.permute(1, 0, 2).reshape(w0 * d * d, Dl * Dr)).reshape(d, d, w2, Dl, Dr)
        x = x.permute(3, 0, 1, 2, 4).reshape(Dl * d * d, w2 * Dr)
        return 1.1 * v + 0.1 * (x @ R2).reshape(v.shape)

    x = b.clone()
    for _ in range(1 if case["prec"] == "fp64" else 6):                # cycles of ten Arnoldi steps
        r = b - apply(x)
        beta = float(r.norm())
        if beta < 1e-15:
            break
        V = [r / beta]
        H = torch.zeros((11, 10), dtype=torch.float64)
        for k in range(10):
            q = apply(V[k])
            for _ in range(2):
                for i in range(k + 1):
                    c = float((V[i] * q).sum())
                    H[i, k] += c
                    q = q - c * V[i]
            H[k + 1, k] = float(q.norm())
            V.append(q / H[k + 1, k])
        rhs = torch.zeros((11, 1), dtype=torch.float64)
        rhs[0, 0] = beta
        y = torch.linalg.lstsq(H, rhs).solution
        for i in range(10):
            x = x + float(y[i, 0]) * V[i]
    return {"x": x}


def _exact_split(case, seed):
    t = _theta(case, seed).cpu().numpy().reshape(case["Dl"] * case["d1"], -1)
    u, s, vt = np.linalg.svd(t, full_matrices=False)
    total = float(np.sum(s * s))
    k = len(s)
    if case["cutoff"] > 0.0:
        tail = np.append(np.cumsum((s * s)[::-1])[::-1], 0.0)
        k = int(next(j for j in range(1, len(s) + 1) if tail[j] <= case["cutoff"] * total))
    k = max(1, min(k, case["chi"]))
    return {"theta": (u[:, :k] * s[:k]) @ vt[:k], "basis": np.eye(k), "sigma": s,
            "disc": float(np.sum(s[k:] ** 2)) / total}


def exact(case, seed):
    if case["kind"] == "evolve":
        return _exact_evolve(case, seed)
    if case["kind"] == "solve":
        return _exact_solve(case, seed)
    if case["kind"] == "split":
        return _exact_split(case, seed)
    return None


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _split_work(m, n, k):
    """A thin SVD (bidiagonalisation, then k vectors of each side)."""
    r, big = min(m, n), max(m, n)
    return {"bytes": 8.0 * (m * n + k * (m + n)), "flops": 4.0 * (big * r * r - r ** 3 / 3.0) + 4.0 * big * r * k}


def _product_work(Dl, Dr, d, w):
    return {"bytes": 8.0 * (w * (Dl * Dl + Dr * Dr) + 2 * Dl * Dr * d * d),
            "flops": 2.0 * w * d * d * Dl * Dr * (Dl + Dr)}


def _sweep_work(L, d, w, chi, products):
    dims = [int(min(chi, float(d) ** i, float(d) ** (L - i))) for i in range(L + 1)]
    total = {"bytes": 0.0, "flops": 0.0}
    for i in range(L - 1):
        a, b = dims[i], dims[i + 2]
        p, s = _product_work(a, b, d, w), _split_work(a * d, d * b, dims[i + 1])
        for key in total:
            total[key] += 2.0 * (products * p[key] + s[key])
    return total


def work(case):
    kind = case["kind"]
    if kind == "evolve":
        steps = math.ceil(math.log(case["tau1"] / case["tau0"]) / math.log(case["ratio"])) + 1
        one = _sweep_work(case["L"], 2, 5, case["chi"], 8)
        return {key: steps * v for key, v in one.items()}
    if kind == "step":
        d, w = (2, 5) if case["model"] == "heisenberg" else (4, 6)
        return _sweep_work(case["L"], d, w, case["chi"], 12)
    if kind == "batch":
        parts = [_sweep_work(L, 2, 5, chi, 12) for L, chi in _batch_sizes(case)]
        return {key: sum(p[key] for p in parts) for key in ("bytes", "flops")}
    if kind == "solve":
        p = _product_work(case["Dl"], case["Dr"], case["d"], case["w"])
        return {"bytes": p["bytes"], "flops": 11.0 * p["flops"]}
    if kind == "split":
        m, n = case["Dl"] * case["d1"], case["d2"] * case["Dr"]
        return _split_work(m, n, min(m, n, case["chi"]))
    dims = [int(min(case["chi"], 2.0 ** i, 2.0 ** (case["L"] - i))) for i in range(case["L"] + 1)]
    flops = sum(4.0 * case["n"] * a * b for a, b in zip(dims, dims[1:]))
    return {"bytes": 8.0 * (sum(2 * a * b for a, b in zip(dims, dims[1:])) + case["L"] * case["n"]), "flops": flops}
