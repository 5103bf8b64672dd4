"""The Krylov kernels at the edges of their dispatch: vector lengths around
those where the threads of the one-workgroup kernels or the number of
workgroups change (1024, 4096 and 8192 entries), bases that fit a thread's
registers, bases beyond (8 vectors) and beyond one pass over 16 vectors, and
a budget of several cycles.

Tolerance: the iterate of a fixed number of GMRES steps is determined to a
small multiple of rounding times the condition of the projected problem
(below 100 here): 1e-10."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from oracle import mps as omps, mpo as ompo
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    c = ite.ite_ctx_create(0)
    yield torch, c
    torch.cuda.synchronize()
    ite.ite_ctx_destroy(c)


@pytest.mark.parametrize("m,cycles", [(3, 2), (10, 1), (20, 1)])
@pytest.mark.parametrize("Dl,Dr", [(3, 7), (16, 16), (17, 16), (32, 32), (33, 32), (45, 45), (64, 32), (64, 33),
                                   (70, 61)])
def test_gmres_iterate_at_length_edges(env, Dl, Dr, m, cycles):
    torch, ctx = env
    rng = np.random.default_rng(Dl * 100 + Dr)
    W = ompo.heisenberg_mpo(4)
    Lm = rng.standard_normal((Dl, 5, Dl)) / np.sqrt(Dl)
    Rm = rng.standard_normal((Dr, 5, Dr)) / np.sqrt(Dr)
    b = rng.standard_normal((Dl, 2, 2, Dr))
    x0 = b + 0.1 * rng.standard_normal(b.shape)
    alpha, beta = 2.5, 0.1
    op = lambda v: alpha * v + beta * omps.heff_apply(Lm, W[1], W[2], Rm, v)
    want, info = omps.gmres(op, b, x0, m, cycles, 0.0)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).cuda()
    x = torch.full(b.shape, np.nan, dtype=torch.float64, device="cuda")
    mv, res = ite.ite_debug_local_solve(ctx, dev(Lm), W[1], W[2], dev(Rm), alpha, beta, dev(b), dev(x0), x,
                                        krylov_dim=m, max_cycles=cycles, tol=0.0)
    assert mv == info["matvecs"]
    got = x.cpu().numpy()
    assert np.max(np.abs(got - want)) <= 1e-10 * np.max(np.abs(want))
    assert abs(res - info["res_rel"]) <= 1e-8 * info["res_rel"] + 1e-14
