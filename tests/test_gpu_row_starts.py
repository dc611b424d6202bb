"""bf16 tiles, one row of them: the k-steps that neighbouring tiles start at depend on how many bytes the rows take.  Every k-step
counts once wherever a tile starts, on both sides of the size where the distance changes.  Operands are small whole numbers, whose
sums are exact: a k-step that is missing, or counted for another, shows at any length."""
import ctypes as C

import pytest

from test_gpu_tiled_tiles import BF16, PART

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(48, 64), (64, 128), (128, 64), (256, 128)], ids="%dx%d".__mod__)
@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("limit", [1 << 20, (4 << 20) // 6 * 5, 4 << 20])
@pytest.mark.parametrize("over", [0, 64])
def test_sums_over_all_of_k(tile, splits, limit, over):
    import torch
    from paper_2502_09922_amd import binding

    fn = binding.lib.ls_test_tiled_gemm
    fn.argtypes = [C.c_uint32] + [C.c_int] * 4 + [C.c_void_p] * 2 + [C.c_int] * 3 + [C.c_void_p] * 2
    bm, bn = tile
    k = limit // (2 * bm) // 64 * 64 + over
    n = 18 * bn + 16  # tiles 0, 8 and 16 share an XCD
    gen = torch.Generator(device="cuda").manual_seed(k)
    a = torch.randint(-3, 4, (bm, k), generator=gen, device="cuda").bfloat16()
    w = torch.randint(-3, 4, (n, k), generator=gen, device="cuda").bfloat16()
    assert 9 * k < 1 << 24
    out = torch.full((splits, bm, n), float("nan"), device="cuda")
    assert fn(BF16, PART, bm, bn, splits, a.data_ptr(), w.data_ptr(), bm, n, k, out.data_ptr(), None)
    assert torch.equal(out.double().sum(0), a.double() @ w.double().T)
