"""The bond split of blocks whose entries, or some of them, are so small that
their squares vanish: whole blocks from 1e-118 down to numbers without a full
mantissa, and blocks of norm one with rows that fall to 1e-250.

Tolerance: as for blocks of ordinary size, 50 eps sqrt(max(m, n)) of the largest
value; where entries have fewer than 53 bits, their last bit (5e-324) as well."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from tests.gpu_util import dev, host
from tests.test_gpu_split import env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def _split(torch, ctx, direction, theta, chi, cutoff):
    m, n = theta.shape
    r = min(m, n)
    A1 = torch.zeros(m * r, dtype=torch.float64, device="cuda")
    A2 = torch.zeros(r * n, dtype=torch.float64, device="cuda")
    k, sig, disc = ite.ite_debug_svd_split(ctx, direction, dev(torch, theta.reshape(m, 1, 1, n)), chi, cutoff, 0.0, A1, A2)
    return k, sig, disc, host(A1)[: m * k].reshape(m, k), host(A2)[: k * n].reshape(k, n)


@pytest.mark.parametrize("direction", [0, 1])
@pytest.mark.parametrize("exponent", [-390, -400, -500, -518, -530, -700, -1000, -1060])
@pytest.mark.parametrize("m,n", [(1, 3), (20, 31), (150, 140), (70, 300), (530, 560)])
def test_tiny_blocks(env, m, n, exponent, direction):  # noqa: F811
    torch, ctx = env
    base = np.random.default_rng(m + n).standard_normal((m, n))
    theta = np.ldexp(base, exponent)
    unit = np.ldexp(theta, -exponent)            # with the bits that theta kept
    k, sig, disc, a1, a2 = _split(torch, ctx, direction, theta, max(1, 2 * min(m, n) // 3), 1e-3)
    s = np.linalg.svd(unit, compute_uv=False)
    tail = np.append(np.cumsum((s * s)[::-1])[::-1], 0.0)
    assert k == min(int(np.argmax(tail <= 1e-3 * tail[0])), max(1, 2 * min(m, n) // 3))
    tol = 50 * np.finfo(float).eps * np.sqrt(max(m, n)) * s[0] + np.ldexp(float(max(m, n)), -1074 - exponent)
    assert np.abs(np.ldexp(sig, -exponent) - s).max() <= tol
    assert abs(disc - tail[k] / tail[0]) <= 1e-12
    if direction == 0:
        basis, prod = a1.T @ a1, a1 @ np.ldexp(a2, -exponent)
    else:
        basis, prod = a2 @ a2.T, np.ldexp(a1, -exponent) @ a2
    assert np.abs(basis - np.eye(k)).max() <= 50 * np.finfo(float).eps * np.sqrt(max(m, n))
    assert np.linalg.norm(unit - prod, 2) <= (s[k] if k < len(s) else 0.0) + tol


@pytest.mark.parametrize("direction", [0, 1])
@pytest.mark.parametrize("size", [24, 60, 150, 260, 530])
@pytest.mark.parametrize("axis", [0, 1])
def test_rows_far_below_the_norm(env, size, direction, axis):  # noqa: F811
    torch, ctx = env
    theta = np.logspace(0, -250, size)[:, None] * np.random.default_rng(size).standard_normal((size, size))
    theta = theta.T.copy() if axis else theta
    k, sig, _, a1, a2 = _split(torch, ctx, direction, theta, size, 0.0)
    s = np.linalg.svd(theta, compute_uv=False)
    tol = 50 * np.finfo(float).eps * np.sqrt(size)
    assert k == size and np.abs(sig - s).max() <= tol * s[0]
    basis = a1.T @ a1 if direction == 0 else a2 @ a2.T
    assert np.abs(basis - np.eye(k)).max() <= tol
    assert np.isfinite(a1).all() and np.isfinite(a2).all()
    assert np.linalg.norm(theta - a1 @ a2, 2) <= tol * s[0]
