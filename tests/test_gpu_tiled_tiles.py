"""Every tile of the tiled GEMM at its own edges, launched with that tile whatever the plan would choose: one row
less and one more than the tile, one more than two tiles, matrices that end inside a tile, K of fewer
k-steps than the ring has stages, with half a k-step at its end, and cut several ways.  Against float64."""
import ctypes as C
import zlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F32, BF16 = 0, 1
PART, STORE, SWIGLU = range(3)
TILES = [(32, 64), (32, 128), (64, 64), (64, 128), (96, 128), (128, 64), (128, 128), (160, 128), (160, 256), (256, 128)]
F32_TILES = TILES[:7] + [(176, 128), (128, 192)]  # 96 x 128 and more: by split operands
CASES = [(F32, t) for t in F32_TILES] + [(BF16, t) for t in TILES]


@pytest.mark.parametrize("dt,tile", CASES, ids=["%s-%dx%d" % (("f32", "bf16")[d], *t) for d, t in CASES])
def test_tile_edges(dt, tile):
    import torch
    from paper_2502_09922_amd import binding

    fn = binding.lib.ls_test_tiled_gemm
    fn.argtypes = [C.c_uint32] + [C.c_int] * 4 + [C.c_void_p] * 2 + [C.c_int] * 3 + [C.c_void_p] * 2
    bm, bn = tile
    tdt, half = (torch.float32, 16) if dt == F32 else (torch.bfloat16, 32)
    gen = torch.Generator().manual_seed(zlib.crc32(b"%d %d %d" % (dt, bm, bn)))
    worst = 0.0
    for m in (bm - 1, bm + 1, 2 * bm + 1):
        for n, k, splits in ((bn + 16, 4 * half, 1), (16, 13 * half, 1), (2 * bn - 16, 41 * half, 1), (bn + 48, 41 * half, 3)):
            for epi in (PART, STORE, SWIGLU):
                if (epi == SWIGLU and bn == 64) or (epi != PART and splits > 1):
                    continue
                rows = n * (2 if epi == SWIGLU else 1)
                a = torch.randn(m, k, generator=gen).to(tdt)
                w = (torch.randn(rows, k, generator=gen) / k**0.5).to(tdt)
                out = torch.full((splits, m, n), float("nan"), dtype=torch.float32 if epi == PART else tdt, device="cuda")
                ad, wd = a.cuda(), w.cuda()
                what = (epi, m, n, k, splits)
                assert fn(dt, epi, bm, bn, splits, ad.data_ptr(), wd.data_ptr(), m, n, k, out.data_ptr(), None), what
                got = out.cpu().double().numpy().sum(0)
                a64, w64 = a.double().numpy(), w.double().numpy()
                z, mag = a64 @ w64.T, np.abs(a64) @ np.abs(w64).T
                err = (k + 8) * 2.0**-23 * mag  # every addition of a sum may lose a last bit of it
                if epi == SWIGLU:
                    g, u, eg, eu = z[:, :n], z[:, n:], err[:, :n], err[:, n:]
                    s = g / (1 + np.exp(-g))
                    z = s * u
                    # |silu'| <= 1.1; the fast exponential and reciprocal: a few last bits, times the exponent
                    err = 1.1 * eg * np.abs(u) + np.abs(s) * eu + eg * eu + (np.abs(g) + 8) * 2.0**-23 * np.abs(z)
                if epi != PART and dt == BF16:
                    err = 1.01 * err + 2.0**-8 * np.abs(z)  # 8 significant bits: half a last bit of [1, 2) is 2^-8
                assert (np.abs(got - z) <= err + 1e-30).all(), (what, np.abs(got - z).max())
                worst = max(worst, float((np.abs(got - z) / err).max()))
    print("largest error %.2f of its bound" % worst)
