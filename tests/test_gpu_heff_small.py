"""H_eff of a small block in one launch: bond dimensions around its 16-wide
tiles, rows per workgroup that do not divide the left bond, MPO bonds from 1 to
16 that differ left and right, rectangular environments, K parts of the last
product that hold no slice, blocks on either side of the rule for the three
launches, and an output that is the input (which takes the three launches).

Tolerance: products and sums of standard normals in FP64, 1e-13 of the largest
entry."""
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


def _run(env, d, w0, w1, w2, Dxl, Dyl, Dxr, Dyr, alias=False):
    torch, ctx = env
    rng = np.random.default_rng(1000 * Dxl + 10 * Dyr + w0 + w2 + d)
    W1 = rng.standard_normal((w0, w1, d, d)) * (rng.random((w0, w1, d, d)) < 0.4)
    W2 = rng.standard_normal((w1, w2, d, d)) * (rng.random((w1, w2, d, d)) < 0.4)
    Lm = rng.standard_normal((Dxl, w0, Dyl))
    Rm = rng.standard_normal((Dxr, w2, Dyr))
    th = rng.standard_normal((Dyl, d, d, Dyr))
    want = omps.heff_apply(Lm, W1, W2, Rm, th)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    square = Dxl == Dyl and Dxr == Dyr
    dt = dev(th)
    y = dt if alias else torch.full((Dxl, d, d, Dxr), np.nan, dtype=torch.float64, device="cuda")
    al = 0.3 if square else 0.0
    ite.ite_debug_heff_apply(ctx, dev(Lm), W1, W2, dev(Rm), dt, al, -0.7, y)
    ref = -0.7 * want + (al * th if square else 0.0)
    assert np.max(np.abs(y.cpu().numpy() - ref)) <= 1e-13 * max(1.0, np.max(np.abs(ref)))


@pytest.mark.parametrize("Dl,Dr", [(1, 1), (1, 2), (2, 1), (3, 4), (4, 3), (15, 17), (16, 16), (17, 15), (31, 33),
                                   (32, 32), (33, 48), (64, 64), (65, 49), (70, 80), (5, 128), (128, 5), (90, 100)])
@pytest.mark.parametrize("d,w", [(2, 5), (4, 6)])
def test_square_blocks(env, d, w, Dl, Dr):
    _run(env, d, w, w, w, Dl, Dl, Dr, Dr)


@pytest.mark.parametrize("d,w0,w1,w2", [(2, 1, 5, 5), (2, 5, 5, 1), (2, 1, 1, 1), (2, 16, 3, 16), (2, 7, 4, 3), (3, 5, 5, 5),
                                        (4, 1, 6, 6), (4, 16, 2, 1), (5, 2, 2, 2)])
@pytest.mark.parametrize("dims", [(7, 5, 9, 6), (20, 33, 18, 34), (1, 8, 40, 3)])
def test_rectangular_blocks(env, d, w0, w1, w2, dims):
    _run(env, d, w0, w1, w2, *dims)


@pytest.mark.parametrize("Dl,Dr", [(3, 4), (20, 32)])
def test_output_over_input(env, Dl, Dr):
    _run(env, 2, 5, 5, 5, Dl, Dl, Dr, Dr, alias=True)
