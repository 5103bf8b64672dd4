"""Blocks of more than 2048 rows and columns, general ones: the bidiagonalisation
step for rows of any length, the ordering of merges in memory and the vectors that
are transformed back in memory, both ways round."""
import numpy as np
import pytest

from tests.test_gpu_split import _check, env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,direction,graded", [(2070, 2055, 0, False), (2055, 2070, 1, True), (2049, 2300, 0, True)])
def test_general_long_blocks(env, m, n, direction, graded):  # noqa: F811
    torch, ctx = env
    rng = np.random.default_rng(m + n)
    theta = rng.standard_normal((m, n))
    if graded:
        r = min(m, n)
        theta = (rng.standard_normal((m, r)) * np.exp(-0.35 * np.log(np.arange(1, r + 1)) ** 2)) @ \
            rng.standard_normal((r, n))
    _check(torch, ctx, direction, theta, 1, 1, 1300)
