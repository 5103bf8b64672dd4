"""The bond split of a block with an entry that is not finite: no singular value
is reported as a number, and a cutoff drops nothing (sizes of every kernel
form, both directions, more rows than columns and the other way round, the bad
entry in the first and last row and column and inside)."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from tests.gpu_util import dev, host
from tests.test_gpu_split import env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("m,n", [(1, 1), (1, 7), (9, 2), (20, 20), (48, 31), (64, 150), (300, 290), (600, 40), (560, 570)])
def test_nonfinite_entry(env, m, n, bad):  # noqa: F811
    torch, ctx = env
    r = min(m, n)
    A1 = torch.zeros(m * r, dtype=torch.float64, device="cuda")
    A2 = torch.zeros(r * n, dtype=torch.float64, device="cuda")
    for i, j in ((0, 0), (m // 2, n // 3), (m - 1, n - 1)):
        theta = np.random.default_rng(m + n).standard_normal((m, n))
        theta[i, j] = bad
        k, sig, _ = ite.ite_debug_svd_split(ctx, i % 2, dev(torch, theta.reshape(m, 1, 1, n)), r, 1e-3, 1e-13, A1, A2)
        assert np.isnan(sig).all()
        assert k == r
        assert not np.isfinite(host(A1)).all() or not np.isfinite(host(A2)).all()
