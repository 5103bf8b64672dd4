"""The bond split where its bidiagonalisation changes from two launches a step
to one (512 rows or columns left) and from there to one workgroup (192 rows),
with one row or column more and less, more rows than columns and the other way
round, and row counts that are no multiple of a workgroup's."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from tests.gpu_util import dev
from tests.test_gpu_split import _check, env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("direction", [0, 1])
@pytest.mark.parametrize("m,n", [(193, 192), (193, 5), (255, 256), (257, 257), (272, 258), (511, 510), (512, 513),
                                 (514, 514), (530, 256), (600, 20), (300, 511)])
def test_split_at_launch_changes(env, direction, m, n):  # noqa: F811
    torch, ctx = env
    rng = np.random.default_rng(2000 * m + n)
    _check(torch, ctx, direction, rng.standard_normal((m, n)), 1, 1, max(1, 2 * min(m, n) // 3))


@pytest.mark.parametrize("size", [30, 100, 190, 250, 400, 520, 700, 1100, 2060])
def test_orthogonal_block(env, size):  # noqa: F811
    # every row is rounding noise once its left reflector has acted: a reflector
    # formed twice from it has to round alike both times
    torch, ctx = env
    rng = np.random.default_rng(size)
    theta, _ = np.linalg.qr(rng.standard_normal((size, size)))
    A1 = torch.zeros(size * size, dtype=torch.float64, device="cuda")
    A2 = torch.zeros(size * size, dtype=torch.float64, device="cuda")
    dt = dev(torch, theta.reshape(size, 1, 1, size))
    k, sig, disc = ite.ite_debug_svd_split(ctx, 0, dt, size, 0.0, 0.0, A1, A2)
    a1, a2, th = A1.view(size, size), A2.view(size, size), dt.view(size, size)
    tol = 50 * np.finfo(float).eps * np.sqrt(size)
    assert k == size and np.abs(sig - 1.0).max() <= tol
    assert float((a1.T @ a1 - torch.eye(size, dtype=torch.float64, device="cuda")).abs().max()) <= tol
    assert float((a1 @ a2 - th).abs().max()) <= tol
