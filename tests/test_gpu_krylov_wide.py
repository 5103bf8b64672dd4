"""One GMRES cycle of up to 64 Krylov vectors, whose steps cross every shape of the
Gram-Schmidt passes, on vectors of one workgroup and of many.

Tolerance: rounding times the condition of the projected problem (10 at 64
steps), as for the shorter cycles: 1e-10."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from oracle import mps as omps
from tests.test_gpu_krylov import env  # noqa: F401  (the fixture)
from tests.test_gpu_krylov_tol import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [17, 20, 25, 33, 64])
@pytest.mark.parametrize("Dl,Dr", [(17, 16), (45, 45), (64, 33), (70, 61), (131, 140)])
def test_wide_basis(env, Dl, Dr, m):  # noqa: F811
    torch, ctx = env
    op, b, x0, args, x = _problem(torch, Dl, Dr, 1.0)
    want, info = omps.gmres(op, b, x0, m, 1, 0.0)
    mv, res = ite.ite_debug_local_solve(ctx, *args, krylov_dim=m, max_cycles=1, tol=0.0)
    assert mv == info["matvecs"] == m + 1
    assert np.max(np.abs(x.cpu().numpy() - want)) <= 1e-10 * np.max(np.abs(want))
    assert abs(res - info["res_rel"]) <= 1e-8 * info["res_rel"] + 1e-14
