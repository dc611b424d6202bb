"""The fp32 tiles by split operands (gemm_split_f32.hip): a value that the parts cannot hold, in the first, a middle and the
last k-step, in a row and in a weight; rows that are cut evenly over tiles, half a k-step at the end.  (Edges and single
products of these tiles: test_gpu_tiled_tiles.py, test_gpu_split_products.py.)"""
import numpy as np
import pytest

from test_gpu_split_products import TILES, matmul

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("where", ["row", "weight"])
@pytest.mark.parametrize("at", [0, 31, 300, 591])
def test_one_value_beyond_the_parts(tile, where, at):
    # 592 = 18.5 k-steps; the largest fp32 value, times weights (or rows) of at most 2^-30
    rng = np.random.default_rng(at)
    m, n, k = 3 * tile[0] + 5, tile[1] + 16, 592
    a, w = rng.standard_normal((m, k)).astype(np.float32), rng.standard_normal((n, k)).astype(np.float32)
    (a if where == "row" else w)[:, at] *= np.float32(2.0**-60)
    (w if where == "row" else a)[:, at] *= np.float32(2.0**-60)
    if where == "row":
        a[m // 2, at] = np.finfo(np.float32).max
    else:
        w[n // 2, at] = np.finfo(np.float32).max
    got = matmul(tile, a, w)
    a64, w64 = a.astype(np.float64), w.astype(np.float64)
    want, mag = a64 @ w64.T, np.abs(a64) @ np.abs(w64).T
    # every addition of a sum may lose a last bit of it, and rounding to fp32 the last one
    assert (np.abs(got - want) <= (k + 8) * 2.0**-23 * mag).all()
