"""The MPO stage inside H_eff at the edges of its column tiles: column counts
below, at and beyond 16, 64 and 256 columns, multiples of four (16-byte loads)
and not, for d = 2 and d = 4, with few and with many workgroups.

Tolerance: products and sums of standard normals in FP64, at most some 1000
terms deep: 1e-13 of the largest entry."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from oracle import mps as omps
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    c = ite.ite_ctx_create(0)
    yield torch, c
    torch.cuda.synchronize()
    ite.ite_ctx_destroy(c)


@pytest.mark.parametrize("d,w", [(2, 5), (4, 6)])
@pytest.mark.parametrize("Dl,Dr", [(1, 1), (3, 4), (2, 15), (5, 16), (4, 17), (3, 60), (2, 64), (2, 68), (3, 257),
                                   (2, 260), (70, 100), (130, 64)])
def test_stage_column_tiles(env, d, w, Dl, Dr):
    torch, ctx = env
    rng = np.random.default_rng(100 * Dl + Dr + d)
    W1 = rng.standard_normal((w, w, d, d)) * (rng.random((w, w, d, d)) < 0.2)
    W2 = rng.standard_normal((w, w, d, d)) * (rng.random((w, w, d, d)) < 0.2)
    Lm = rng.standard_normal((Dl, w, Dl))
    Rm = rng.standard_normal((Dr, w, Dr))
    th = rng.standard_normal((Dl, d, d, Dr))
    want = omps.heff_apply(Lm, W1, W2, Rm, th)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    y = torch.full((Dl, d, d, Dr), np.nan, dtype=torch.float64, device="cuda")
    ite.ite_debug_heff_apply(ctx, dev(Lm), W1, W2, dev(Rm), dev(th), 0.0, 1.0, y)
    assert np.max(np.abs(y.cpu().numpy() - want)) <= 1e-13 * max(1.0, np.max(np.abs(want)))
