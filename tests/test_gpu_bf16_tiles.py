"""The bf16 tiles of the tiled GEMM that its own test does not name, at their edges: rows that are not fetched in the last
tile of a column, columns that are not fetched in the last panel, fewer k-steps than the ring has stages, half a k-step
at the end, K cut several ways, and one tile row (k-steps in cyclic order, another start for each tile).  Against
float64."""
import ctypes as C

import pytest

from test_gpu_tiled_tiles import BF16, PART, STORE, test_tile_edges as edges

pytestmark = pytest.mark.gpu

GLU = [(32, 96), (48, 96), (64, 96), (64, 224), (96, 192), (128, 192), (160, 192), (256, 192)]
PLAIN = [(48, 48), (48, 64), (64, 48), (96, 96), (128, 96), (160, 96)]


@pytest.mark.parametrize("tile", GLU, ids="%dx%d".__mod__)
def test_tile_edges(tile):
    edges(BF16, tile)


@pytest.mark.parametrize("tile", PLAIN + GLU, ids="%dx%d".__mod__)
def test_rows_and_columns_that_are_not_fetched(tile):
    import torch
    from paper_2502_09922_amd import binding

    fn = binding.lib.ls_test_tiled_gemm
    fn.argtypes = [C.c_uint32] + [C.c_int] * 4 + [C.c_void_p] * 2 + [C.c_int] * 3 + [C.c_void_p] * 2
    bm, bn = tile
    gen = torch.Generator().manual_seed(1000 * bm + bn)
    for m in (1, bm - 15, bm, bm + 1, 2 * bm + 9):
        for n, k, splits in ((bn + 16, 64, 1), (16, 13 * 32, 1), (9 * bn - 16, 20 * 64, 1), (3 * bn + 16, 20 * 64, 3), (3 * bn, 41 * 32, 3)):
            a = torch.randn(m, k, generator=gen).to(torch.bfloat16)
            w = (torch.randn(n, k, generator=gen) / k**0.5).to(torch.bfloat16)
            z, mag = a.double() @ w.double().T, a.double().abs() @ w.double().abs().T
            for epi in (PART, STORE)[: 1 if splits > 1 else 2]:
                out = torch.full((splits, m, n), float("nan"), dtype=torch.float32 if epi == PART else torch.bfloat16, device="cuda")
                ad, wd = a.cuda(), w.cuda()
                what = (epi, m, n, k, splits)
                assert fn(BF16, epi, bm, bn, splits, ad.data_ptr(), wd.data_ptr(), m, n, k, out.data_ptr(), None), what
                # every addition of a sum may lose a last bit of it; then 8 significant bits: half a last bit of [1, 2) is 2^-8
                err = (k + 8) * 2.0**-23 * mag
                if epi == STORE:
                    err = 1.01 * err + 2.0**-8 * z.abs()
                assert ((out.cpu().double().sum(0) - z).abs() <= err + 1e-30).all(), what
