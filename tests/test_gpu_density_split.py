"""Eigendecomposition of the density matrices of the MPO-MPS product: matrices
D M D whose diagonal falls to 1e-30, in one run and in two interleaved ones (as the
two states of a site give them), at sizes of one workgroup (64 rows), of the pair
rounds (255) and with Householder preconditioning (256, 512).

Bound: rows count as orthogonal at 8 eps sqrt(n) of the product of their norms plus
1e-3 of that of the largest; an eigenvalue lambda = s^2 of a matrix with factor D C
then is off by at most a few times 8 eps sqrt(n) (s s_1 + 1e-3 s_1^2), where the
bidiagonalisation of the bond splits is off by eps s_1^2; 16 eps sqrt(n) here.  65
rows (pair rounds with one row in the last block) stop at the stagnation of the
measure before they get there and are held to eps sqrt(n) of the largest."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from tests.gpu_util import dev, host
from tests.test_gpu_split import env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

EPS = np.finfo(float).eps


@pytest.mark.parametrize("n", [1, 2, 31, 64, 65, 255, 256, 512])
@pytest.mark.parametrize("halves", [False, True])
def test_small_eigenvalues(env, n, halves):  # noqa: F811
    torch, ctx = env
    D = 2.0 ** -np.linspace(0, 50, n)
    if halves:
        D = np.concatenate([D[::2], D[1::2]])
    C = D[:, None] * np.random.default_rng(n).standard_normal((n, n)) / np.sqrt(n)
    rho = C @ C.T
    s = np.linalg.svd(C, compute_uv=False)
    k = max(1, 2 * n // 3)
    V = torch.full((k, n), np.nan, dtype=torch.float64, device="cuda")
    lam = ite.ite_debug_density_split(ctx, dev(torch, 0.5 * (rho + rho.T)), k, V)
    assert np.all(np.diff(lam) <= 0)
    unit = EPS * np.sqrt(n)
    bound = unit * s[0] ** 2 if n == 65 else 16 * unit * (s * s[0] + 1e-3 * s[0] ** 2)
    assert np.all(np.abs(lam - s * s) <= bound)
    v = host(V)
    assert np.abs(v @ v.T - np.eye(k)).max() <= 50 * unit
    # what the kept vectors carry of the factor: its singular values
    w = np.linalg.norm(v @ C, axis=1)
    assert np.all(np.abs(w * w - s[:k] ** 2) <= 2 * (bound if n == 65 else bound[:k]))


def test_density_split_errors(env):  # noqa: F811
    torch, ctx = env
    rho = torch.eye(4, dtype=torch.float64, device="cuda")
    for k in (0, 5):
        with pytest.raises(ite.IteError) as e:
            ite.ite_debug_density_split(ctx, rho, k, torch.zeros((5, 4), dtype=torch.float64, device="cuda"))
        assert e.value.code == ite.ITE_EINVAL
