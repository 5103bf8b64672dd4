"""Tolerance-driven GMRES, whose columns come to the host through the mailbox while
the next step is already issued: vector lengths around those where the kernels
change, restarts, bases of more than 16 vectors, and solves that end while a
step nobody needs is under way, one after the other without a wait.

The tolerances lie at least 5% off every residual on the way (on the CPU), so the
number of products is determined.  Iterates: rounding times the condition of the
projected problem (below 100), 1e-10; refined solutions: the residual target times
the condition of the operator (below 10)."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from oracle import mps as omps, mpo as ompo
from tests.test_gpu_krylov import env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

SIZES = [(3, 7), (16, 16), (17, 16), (32, 32), (33, 32), (45, 45), (64, 32), (64, 33), (70, 61)]


def _problem(torch, Dl, Dr, beta):
    rng = np.random.default_rng(Dl * 100 + Dr)
    W = ompo.heisenberg_mpo(4)
    Lm = rng.standard_normal((Dl, 5, Dl)) / np.sqrt(Dl)
    Rm = rng.standard_normal((Dr, 5, Dr)) / np.sqrt(Dr)
    b = rng.standard_normal((Dl, 2, 2, Dr))
    x0 = b + 0.1 * rng.standard_normal(b.shape)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda()
    op = lambda v: 2.5 * v + beta * omps.heff_apply(Lm, W[1], W[2], Rm, v)
    x = torch.full(b.shape, np.nan, dtype=torch.float64, device="cuda")
    return op, b, x0, (dev(Lm), W[1], W[2], dev(Rm), 2.5, beta, dev(b), dev(x0), x), x


@pytest.mark.parametrize("m,cycles,beta,tol", [(4, 12, 0.1, 1.5e-8), (4, 12, 0.1, 1e-11), (24, 2, 0.6, 2e-7),
                                               (10, 1, 0.1, 0.5)])
@pytest.mark.parametrize("Dl,Dr", SIZES)
def test_iterate_and_products(env, Dl, Dr, m, cycles, beta, tol):  # noqa: F811
    torch, ctx = env
    op, b, x0, args, x = _problem(torch, Dl, Dr, beta)
    want, info = omps.gmres(op, b, x0, m, cycles, tol)
    for _ in range(2):
        x.fill_(np.nan)
        mv, res = ite.ite_debug_local_solve(ctx, *args, krylov_dim=m, max_cycles=cycles, tol=tol)
        assert mv == info["matvecs"]
        assert np.max(np.abs(x.cpu().numpy() - want)) <= 1e-10 * np.max(np.abs(want))
        assert abs(res - info["res_rel"]) <= 1e-8 * info["res_rel"] + 1e-14


@pytest.mark.parametrize("precision", [ite.PREC_FP32_IR, ite.PREC_BF16_IR])
@pytest.mark.parametrize("Dl,Dr", SIZES)
def test_solves_in_a_row_with_a_step_under_way(env, Dl, Dr, precision):  # noqa: F811
    # every correction ends after its first step, the second already issued
    torch, ctx = env
    op, b, x0, args, x = _problem(torch, Dl, Dr, 0.1)
    mv, res = ite.ite_debug_local_solve(ctx, *args, krylov_dim=10, max_cycles=1, tol=0.5, precision=precision,
                                        max_refine=40, tol_refine=1e-10)
    assert res <= 1e-10
    want, _ = omps.gmres(op, b, x0, 24, 4, 1e-13)
    assert np.linalg.norm(x.cpu().numpy() - want) <= 1e-9 * np.linalg.norm(want)
    r = b - op(x.cpu().numpy())
    assert abs(np.linalg.norm(r) / np.linalg.norm(b) - res) <= 1e-13
