"""The bond split where its bidiagonalisation changes from two launches a step
to one (512 rows or columns left) and from there to one workgroup (192 rows),
with one row or column more and less, more rows than columns and the other way
round, and row counts that are no multiple of a workgroup's."""
import numpy as np
import pytest

from tests.test_gpu_split import _check, env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("direction", [0, 1])
@pytest.mark.parametrize("m,n", [(193, 192), (193, 5), (255, 256), (257, 257), (272, 258), (511, 510), (512, 513),
                                 (514, 514), (530, 256), (600, 20), (300, 511)])
def test_split_at_launch_changes(env, direction, m, n):  # noqa: F811
    torch, ctx = env
    rng = np.random.default_rng(2000 * m + n)
    _check(torch, ctx, direction, rng.standard_normal((m, n)), 1, 1, max(1, 2 * min(m, n) // 3))
