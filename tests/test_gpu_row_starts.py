"""bf16 tiles, one row of them: the k-steps that neighbouring tiles start at depend on how many bytes the rows take.  Every k-step
counts once wherever a tile starts, at and just above the sizes where the distance changes.  Against float64."""
import ctypes as C

import pytest

from test_gpu_tiled_tiles import BF16, PART

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(48, 64), (64, 128), (128, 64), (256, 128)], ids="%dx%d".__mod__)
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("limit,over", [(20, 0), (20, 64), (22, 0), (22, 64)])
def test_sums_over_all_of_k(tile, splits, limit, over):
    import torch
    from paper_2502_09922_amd import binding

    fn = binding.lib.ls_test_tiled_gemm
    fn.argtypes = [C.c_uint32] + [C.c_int] * 4 + [C.c_void_p] * 2 + [C.c_int] * 3 + [C.c_void_p] * 2
    bm, bn = tile
    k = (1 << limit) // (2 * bm) // 64 * 64 + over
    n = 18 * bn + 16  # tiles 0, 8 and 16 share an XCD
    gen = torch.Generator(device="cuda").manual_seed(k)
    a = torch.randn(bm, k, generator=gen, device="cuda").bfloat16()
    w = (torch.randn(n, k, generator=gen, device="cuda") / k**0.5).bfloat16()
    z, mag = a.double() @ w.double().T, a.double().abs() @ w.double().abs().T
    out = torch.full((splits, bm, n), float("nan"), device="cuda")
    assert fn(BF16, PART, bm, bn, splits, a.data_ptr(), w.data_ptr(), bm, n, k, out.data_ptr(), None)
    # every addition of a sum may lose a last bit of it
    assert ((out.double().sum(0) - z).abs() <= (k + 8) * 2.0**-23 * mag).all()
