"""Large outputs of short products: K up to 128 takes 64 x 64 tiles with one K part,
alone and in a grouped launch, more takes two; FP32 takes larger tiles from a K
of 512 on.

Tolerances: those of the products at tile edges; a step whose first contraction
has such a shape is the same alone and in a batch to the rounding of its
reductions (1e-12 in the energy)."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from paper_2606_02930_amd import hamiltonians
from tests.gpu_util import mps_overlap
from tests.test_gpu_gemm_tiles import _run, env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", [(2113, 2050, 1), (2113, 2050, 16), (2050, 2113, 17), (2113, 2050, 128),
                                   (2050, 2113, 129), (1100, 2017, 127), (66000, 32, 5), (33, 66000, 64),
                                   (2900, 2950, 511), (2900, 2950, 512)])
def test_short_products(env, shape, tA, tB):  # noqa: F811
    _run(env, shape, tA, tB, 0, 1e-13)
    _run(env, shape, tA, tB, 1, 6e-6)


# one full round of 64 x 64 tiles and a few tiles more, with a long K
@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", [(1024, 2048, 1024), (1000, 2040, 1503), (500, 4070, 1031), (1025, 2048, 1031)])
def test_one_round_of_long_products(env, shape, tA, tB):  # noqa: F811
    _run(env, shape, tA, tB, 0, 1e-13)


@pytest.mark.parametrize("precision", [ite.PREC_FP64, ite.PREC_FP32_IR])
def test_short_first_contraction_in_a_batch(env, precision):  # noqa: F811
    # d = 4: the block between bonds of 64 and 600 is 384 x 9600 with K = 64
    torch, ctx = env
    dims = [1, 4, 16, 64, 160, 600, 256, 64, 16, 4, 1]
    L, rng = len(dims) - 1, np.random.default_rng(7)
    A, carry = [None] * L, np.ones((1, 1))
    for i in range(L - 1, 0, -1):
        a = np.tensordot(rng.standard_normal((dims[i], 4, dims[i + 1])), carry, axes=([2], [0])).reshape(dims[i], -1)
        q, r = np.linalg.qr(a.T)
        A[i], carry = np.ascontiguousarray(q.T).reshape(dims[i], 4, -1), r.T / np.linalg.norm(r)
    A[0] = np.tensordot(rng.standard_normal((1, 4, 4)), carry, axes=([2], [0]))
    A[0] /= np.linalg.norm(A[0])
    H = ite.ite_mpo_load(ctx, hamiltonians.anderson_star(4.0, -2.0, np.linspace(-1, 1, L - 1), np.full(L - 1, 0.25)))
    o = ite.ite_default_opts(chi_max=600, cutoff=0.0, precision=precision, max_refine=2 if precision else 0,
                             krylov_dim=4)
    psi = [ite.ite_mps_load(ctx, A, 600) for _ in range(3)]
    try:
        alone = ite.ite_imag_step(ctx, psi[0], H, 0.02, o)
        both, status = ite.ite_step_batch(ctx, psi[1:], [H, H], [0.02, 0.02], [o, o])
        assert status == [0, 0] and both[0]["energy"] == both[1]["energy"]
        assert abs(both[0]["energy"] - alone["energy"]) <= 1e-12 * abs(alone["energy"])
        x, y = (ite.ite_mps_export(ctx, p, [4] * L) for p in psi[:2])
        assert abs(abs(mps_overlap(x, y)) - 1.0) <= 1e-12
    finally:
        for p in psi:
            ite.ite_mps_destroy(p)
        ite.ite_mpo_destroy(H)
