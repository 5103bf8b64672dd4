"""GPU products at the edges of their tiles: 16, 32 and 64 wide workgroup tiles
with remainders in every direction, sides too short for a wide side-contiguous
tile, K shorter than a slice, and K split over workgroups.  The operands sit in
wider buffers filled with NaN, so a value read from outside the matrix shows.

Tolerances: FP64 sums of K products differ from numpy's by at most a few
sqrt(K) eps of the largest entry (K = 8192: 2e-14 x 4); FP32 accumulation (FP32
operands, or BF16 operands rounded beforehand) by sqrt(K) 2^-24 for K terms in
a row (K = 500, or K = 8192 in eight parts or more: below 2e-6 x 3).
"""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

F64 = [(1, 1, 1), (16, 16, 16), (17, 31, 15), (33, 16, 511), (15, 33, 513),     # 16 wide
       (700, 300, 500), (500, 417, 33), (6200, 31, 40), (31, 6200, 40),         # 32 wide, sides below 32
       (2100, 1100, 77), (1472, 1537, 128),                                     # 64 wide
       (40, 33, 8192), (17, 5, 8192), (33, 17, 4112)]                           # K over workgroups
F32 = [(1, 1, 1), (33, 31, 15), (65, 129, 500), (700, 300, 500), (500, 417, 33), (6200, 31, 40), (31, 6200, 40),
       (2100, 2050, 50), (40, 33, 8192)]
BF16 = [(1, 1, 1), (17, 33, 63), (33, 17, 64), (65, 129, 500), (700, 300, 500), (500, 417, 65), (6200, 31, 40),
        (31, 6200, 40), (2050, 2040, 130), (2900, 2950, 33)]


@pytest.fixture(scope="module")
def env():
    torch = require_gpu()
    c = ite.ite_ctx_create(0)
    yield torch, c
    torch.cuda.synchronize()
    ite.ite_ctx_destroy(c)


def _run(env, shape, tA, tB, prec, tol):
    torch, ctx = env
    M, N, K = shape
    rng = np.random.default_rng(M + 3 * N + 7 * K + 2 * tA + tB)

    def operand(rows, cols, pad):
        x = rng.standard_normal((rows, cols))
        if prec == 1:
            x = x.astype(np.float32).astype(np.float64)
        elif prec == 2:
            m, e = np.frexp(x)
            x = np.ldexp(np.round(m * 256.0) / 256.0, e)
        buf = np.full((rows, cols + pad), np.nan)
        buf[:, :cols] = x
        return x, torch.from_numpy(buf).cuda(), cols + pad

    A, dA, lda = operand(*((K, M) if tA else (M, K)), 3)
    B, dB, ldb = operand(*((N, K) if tB else (K, N)), 1)
    C = rng.standard_normal((M, N))
    dD = torch.full((M, N + 2), 7.0, dtype=torch.float64, device="cuda")
    dD[:, :N] = torch.from_numpy(C).cuda()
    ite.ite_debug_gemm(ctx, tA, tB, M, N, K, 0.7, dA, lda, dB, ldb, -1.3, dD, N + 2, dD, N + 2, prec)
    want = 0.7 * ((A.T if tA else A) @ (B.T if tB else B)) - 1.3 * C
    got = dD.cpu().numpy()
    assert np.all(got[:, N:] == 7.0)
    assert np.max(np.abs(got[:, :N] - want)) <= tol * max(1.0, np.max(np.abs(want)))


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", F64)
def test_fp64_product_at_tile_edges(env, shape, tA, tB):
    _run(env, shape, tA, tB, 0, 1e-13)


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", F32)
def test_fp32_product_at_tile_edges(env, shape, tA, tB):
    _run(env, shape, tA, tB, 1, 6e-6)


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", BF16)
def test_bf16_product_at_tile_edges(env, shape, tA, tB):
    _run(env, shape, tA, tB, 2, 6e-6)


# tiles larger than 64 x 64, from 1024 of those on with a K of 1024 or more, or 2048 in
# FP32: their remainders in both directions and in K, and sides shorter than one
# wavefront tile, which keep the 64 x 64
LARGE = [(2100, 2020, 1024), (1985, 2113, 1031), (3000, 2800, 77), (65600, 33, 1025), (33, 65600, 1025),
         (131100, 64, 33), (65, 66000, 1040)]


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", LARGE)
def test_large_tiles(env, shape, tA, tB):
    _run(env, shape, tA, tB, 0, 1e-13)
    _run(env, shape, tA, tB, 1, 6e-6)
