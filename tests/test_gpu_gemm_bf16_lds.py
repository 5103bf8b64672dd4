"""BF16 products on either side of the rule for the tiles staged through LDS, with
rows that allow 16-byte loads and rows that do not: 256 tiles and more, 160 with
a long K, 128 with a K shorter than a slice.  Rows are padded with NaN.

Tolerance: products of BF16 values are exact in FP32; a chain of K additions of
standard normals is off by about 2^-24 K of a largest sum of 5 sqrt(K), 5 of its
standard deviations over all entries: below 6e-6 of the largest entry for
K = 2056."""
import numpy as np
import pytest

import paper_2606_02930_amd as ite
from tests.test_gpu_gemm_tiles import env  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", [(2040, 2056, 264), (2056, 1032, 40), (1928, 1536, 2056), (2048, 1024, 264), (1536, 4088, 72)])
@pytest.mark.parametrize("align", [8, 1])
def test_bf16_product_around_the_rule(env, shape, tA, tB, align):  # noqa: F811
    torch, ctx = env
    M, N, K = shape
    g = torch.Generator(device="cuda").manual_seed(M + N + K)

    def operand(rows, cols):
        x = torch.randn((rows, cols), dtype=torch.float64, device="cuda", generator=g).bfloat16().double()
        buf = torch.full((rows, cols + align), float("nan"), dtype=torch.float64, device="cuda")
        buf[:, :cols] = x
        return x, buf, cols + align

    A, dA, lda = operand(*((K, M) if tA else (M, K)))
    B, dB, ldb = operand(*((N, K) if tB else (K, N)))
    C = torch.randn((M, N), dtype=torch.float64, device="cuda", generator=g)
    D = torch.full((M, N + 2), 7.0, dtype=torch.float64, device="cuda")
    D[:, :N] = C
    ite.ite_debug_gemm(ctx, tA, tB, M, N, K, 0.7, dA, lda, dB, ldb, -1.3, D, N + 2, D, N + 2, 2)
    want = 0.7 * ((A.T if tA else A) @ (B.T if tB else B)) - 1.3 * C
    assert bool((D[:, N:] == 7.0).all())
    assert float((D[:, :N] - want).abs().max()) <= 6e-6 * float(want.abs().max())
