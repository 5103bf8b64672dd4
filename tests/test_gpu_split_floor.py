"""Vanishing and very small singular values of a block: rank 3, and values that
fall to 1e-16 of the largest, at sizes of one and of several merge levels.

Tolerance: the bidiagonalisation and the merges round at eps of the largest
value; 4 eps leaves room for a few such roundings (8 eps, the deflation of
values of the size of the largest, is too coarse here)."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from tests.gpu_util import dev
from tests.test_gpu_split import env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

EPS = np.finfo(float).eps


@pytest.mark.parametrize("size", [12, 33, 64, 150, 300, 520])
@pytest.mark.parametrize("values", ["rank3", "small"])
def test_small_values_keep_their_place(env, size, values):  # noqa: F811
    torch, ctx = env
    rng = np.random.default_rng(size)
    u, _ = np.linalg.qr(rng.standard_normal((size, size)))
    v, _ = np.linalg.qr(rng.standard_normal((size, size)))
    s = np.where(np.arange(size) < 3, 1.0, 0.0) if values == "rank3" else np.logspace(0, -16, size)
    th = dev(torch, ((u * s) @ v).reshape(size, 1, 1, size))
    A1 = torch.zeros(size * size, dtype=torch.float64, device="cuda")
    A2 = torch.zeros(size * size, dtype=torch.float64, device="cuda")
    _, sig, _ = ite.ite_debug_svd_split(ctx, 0, th, size, 0.0, 0.0, A1, A2)
    assert np.abs(sig - s)[s < 1e-14].max() <= 4 * EPS
    if values == "rank3":
        k, _, _ = ite.ite_debug_svd_split(ctx, 0, th, size, 1e-30, 0.0, A1, A2)
        assert k == 3
