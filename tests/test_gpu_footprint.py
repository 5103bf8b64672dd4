"""The admission estimate of the server covers what a request takes on the device:
peak of a context's allocations over one step, in FP64 and with FP32 shadows,
for blocks beyond 2048 rows (whose vectors are transformed back in memory) and
below."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from paper_2606_02930_amd import hamiltonians
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def _chain(L, d):
    if d == 2:
        return hamiltonians.heisenberg(L)
    A = np.diag(np.arange(d) / (4.0 * d))
    W = np.zeros((3, 3, d, d))
    W[0, 0] = W[2, 2] = np.eye(d)
    W[0, 1] = W[1, 2] = A
    W[0, 2] = 0.1 * A
    return [W[:1].copy()] + [W.copy() for _ in range(L - 2)] + [W[:, 2:].copy()]


@pytest.mark.parametrize("precision", [ite.PREC_FP64, ite.PREC_FP32_IR])
@pytest.mark.parametrize("L,d,chi", [(8, 8, 300), (20, 2, 300)])
@pytest.mark.parametrize("batch", [False, True])
def test_estimate_covers_a_step(L, d, chi, precision, batch):
    torch = require_gpu()
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    base = torch.cuda.memory_allocated()
    ctx = ite.ite_ctx_create(0)
    Ws = _chain(L, d)
    rng = np.random.default_rng(L)
    H = ite.ite_mpo_load(ctx, Ws)
    psi = ite.ite_mps_create(ctx, [x / np.linalg.norm(x) for x in rng.standard_normal((L, d))], chi, pad_full=True)
    o = ite.ite_default_opts(chi_max=chi, cutoff=0.0, precision=precision)
    if batch:
        ite.ite_step_batch(ctx, [psi], [H], [0.05], [o])
    else:
        ite.ite_imag_step(ctx, psi, H, 0.05, o)
    peak = torch.cuda.max_memory_allocated() - base
    ite.ite_mps_destroy(psi)
    ite.ite_mpo_destroy(H)
    ite.ite_ctx_destroy(ctx)
    assert peak <= ite.ite_request_footprint([d] * L, [1] + [w.shape[1] for w in Ws], chi, o.krylov_dim)
