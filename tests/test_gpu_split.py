"""The bond split by bidiagonalisation and divide and conquer at the sizes
where its kernels change: one and two columns, the last size done by one
workgroup and the first that is merged (32, 33 rows), chunk and register
limits of the reflector launches (128, 512 rows), one row more than the
longest vector held in registers (2048), and spectra that deflate almost
everything (equal, grouped and vanishing singular values)."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from tests.gpu_util import require_gpu, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    ctx = ite.ite_ctx_create(0)
    yield torch, ctx
    torch.cuda.synchronize()
    ite.ite_ctx_destroy(ctx)


def _check(torch, ctx, direction, theta, d1, d2, chi):
    m, n = theta.shape
    r = min(m, n)
    A1 = torch.zeros(m * r, dtype=torch.float64, device="cuda")
    A2 = torch.zeros(r * n, dtype=torch.float64, device="cuda")
    k, sig, disc = ite.ite_debug_svd_split(ctx, direction, dev(torch, theta.reshape(m // d1, d1, d2, n // d2)), chi,
                                           0.0, 0.0, A1, A2)
    u, s, vt = np.linalg.svd(theta, full_matrices=False)
    assert k == min(r, chi)
    # backward-stable in both: a few eps sqrt(mn) of the largest value
    tol = 50 * np.finfo(float).eps * np.sqrt(max(m, n))
    assert np.abs(sig - s).max() <= tol * s[0]
    a1, a2 = host(A1)[: m * k].reshape(m, k), host(A2)[: k * n].reshape(k, n)
    basis = a1.T @ a1 if direction == 0 else a2 @ a2.T
    assert np.abs(basis - np.eye(k)).max() <= tol
    # the rest has the norm of the dropped values
    assert np.linalg.norm(theta - a1 @ a2, 2) <= (s[k] if k < r else 0.0) + tol * s[0]


@pytest.mark.parametrize("direction", [0, 1])
@pytest.mark.parametrize("m,n", [(1, 40), (40, 2), (33, 33), (34, 65), (66, 64), (130, 128), (129, 7), (512, 96),
                                 (514, 130), (96, 2050)])
def test_split_sizes(env, direction, m, n):
    torch, ctx = env
    rng = np.random.default_rng(1000 * m + n)
    _check(torch, ctx, direction, rng.standard_normal((m, n)), 1, 1, max(1, 2 * min(m, n) // 3))


@pytest.mark.parametrize("size", [33, 64, 150, 300])
@pytest.mark.parametrize("values", ["equal", "groups", "rank3", "decades", "diagonal", "tiny"])
def test_split_deflating_spectra(env, size, values):
    torch, ctx = env
    rng = np.random.default_rng(size)
    u, _ = np.linalg.qr(rng.standard_normal((size, size)))
    v, _ = np.linalg.qr(rng.standard_normal((size, size)))
    s = {"equal": np.ones(size), "groups": np.repeat(2.0 ** -np.arange(size // 3 + 1.0), 3)[:size],
         "rank3": np.where(np.arange(size) < 3, 1.0, 0.0), "decades": np.logspace(0, -40, size),
         "diagonal": np.linspace(1, 2, size), "tiny": np.full(size, 1e-120)}[values]
    theta = np.diag(s) if values == "diagonal" else (u * s) @ v
    _check(torch, ctx, 0, theta, 1, 1, size)


def test_split_of_zero_and_of_nan(env):
    torch, ctx = env
    n = 70
    A1 = torch.zeros(n * n, dtype=torch.float64, device="cuda")
    A2 = torch.zeros(n * n, dtype=torch.float64, device="cuda")
    k, sig, _ = ite.ite_debug_svd_split(ctx, 0, dev(torch, np.zeros((n, 1, 1, n))), n, 0.0, 0.0, A1, A2)
    assert k == n and np.all(sig == 0.0)
    a1 = host(A1).reshape(n, n)
    assert np.abs(a1.T @ a1 - np.eye(n)).max() < 1e-13
    bad = np.ones((n, n))
    bad[3, 5] = np.nan
    ite.ite_debug_svd_split(ctx, 0, dev(torch, bad.reshape(n, 1, 1, n)), n, 0.0, 0.0, A1, A2)
    assert not np.isfinite(host(A1)).all() or not np.isfinite(host(A2)).all()
