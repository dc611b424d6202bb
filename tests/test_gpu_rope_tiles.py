"""RoPE and the cache append in the tiled GEMM's epilogue.  Every tile there is, launched by name: one to eight row blocks of a
wavefront, row positions loaded before the products and behind them, table entries a row block ahead and not; last row
blocks that are not full, heads that end inside a tile, rows of one sequence beside another's, rows without room.  Against
float64.  Then prompts through a stage, and the generation step behind them, which reads what was appended."""
import ctypes as C

import pytest

import synth
from test_gpu_tiled_gemm import run

pytestmark = pytest.mark.gpu

F32, BF16 = 0, 1
BF16_TILES = [(32, 64), (32, 96), (32, 128), (48, 48), (48, 64), (48, 96), (64, 48), (64, 64), (64, 96), (64, 128), (64, 224),
              (96, 96), (96, 128), (96, 192), (128, 64), (128, 96), (128, 128), (128, 192), (160, 96), (160, 128), (160, 192),
              (160, 256), (256, 128), (256, 192)]
F32_TILES = [(32, 64), (32, 128), (64, 64), (64, 128), (128, 64), (96, 128), (128, 128), (176, 128), (128, 192)]


@pytest.mark.parametrize("heads", [(3, 2, 64), (2, 1, 128)], ids="%d+%dx%d".__mod__)
@pytest.mark.parametrize("dt,tile", [(BF16, t) for t in BF16_TILES] + [(F32, t) for t in F32_TILES],
                         ids=["%s-%dx%d" % (("f32", "bf16")[d], *t) for d, t in [(BF16, t) for t in BF16_TILES] + [(F32, t) for t in F32_TILES]])
def test_chosen_tile(dt, tile, heads):
    import torch
    from paper_2502_09922_amd import binding

    fn = binding.lib.ls_test_tiled_rope
    fn.argtypes = [C.c_uint32] + [C.c_int] * 2 + [C.c_void_p] * 2 + [C.c_int] * 2 + [C.c_void_p] * 4 + [C.c_int] * 4 + [C.c_void_p] * 3
    (bm, bn), (hq, hkv, hd) = tile, heads
    tdt, k, seqs, room = (torch.float32, 112, 3, 300) if dt == F32 else (torch.bfloat16, 416, 3, 300)
    n = (hq + 2 * hkv) * hd
    gen = torch.Generator().manual_seed(1000 * bm + bn + hd)
    angle = torch.arange(room, dtype=torch.float64)[:, None] * 10000.0 ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64) / hd)
    table = torch.stack([angle.cos(), angle.sin()], -1).float()
    for m in (1, bm - 1, bm + 17, 2 * bm + 1):
        a = torch.randn(m, k, generator=gen).to(tdt)
        w = (torch.randn(n, k, generator=gen) / k**0.5).to(tdt)
        seq = torch.arange(m, dtype=torch.int32) * seqs // m
        pos = torch.zeros(m, dtype=torch.int32)
        for s in range(seqs):
            pos[seq == s] = torch.randperm(room, generator=gen)[: int((seq == s).sum())].int()
        pos[5::29] = -1  # no room left
        out = torch.full((m, n), float("nan"), dtype=tdt, device="cuda")
        kc, vc = (torch.full((seqs, hkv, room, hd), float("nan"), dtype=tdt, device="cuda") for _ in range(2))
        dev = [t.cuda() for t in (a, w, table, seq, pos)]
        assert fn(dt, bm, bn, dev[0].data_ptr(), dev[1].data_ptr(), m, k, out.data_ptr(), dev[2].data_ptr(), dev[3].data_ptr(),
                  dev[4].data_ptr(), hq, hkv, hd, room, kc.data_ptr(), vc.data_ptr(), None), (tile, m)
        out, kc, vc = out.cpu().double(), kc.cpu().double(), vc.cpu().double()
        z, mag = a.double() @ w.double().T, a.double().abs() @ w.double().abs().T
        err = (k + 8) * 2.0**-23 * mag  # every addition of a sum may lose a last bit of it
        u = 2.0**-8 if dt == BF16 else 2.0**-22  # of a stored bf16 value; of the rotation's fp32 products and sum
        if dt == BF16:
            err = 1.01 * err + u * z.abs()  # the projection is rounded before it turns
        z, err = z.view(m, -1, hd), err.view(m, -1, hd)
        live = pos >= 0
        cs = table.double()[pos.clamp(min=0).long()][:, None]
        c, s = cs[..., 0], cs[..., 1]
        turned = torch.stack([z[..., 0::2] * c - z[..., 1::2] * s, z[..., 0::2] * s + z[..., 1::2] * c], -1).reshape(z.shape)
        both = (err[..., 0::2] + err[..., 1::2]).repeat_interleave(2, -1)
        size = (z[..., 0::2].abs() + z[..., 1::2].abs()).repeat_interleave(2, -1)
        bound = 1.01 * both + u * (turned.abs() if dt == BF16 else size) + 2.0**-22 * size
        got_q, got = out.view(m, -1, hd)[:, :hq], (out.view(m, -1, hd), kc, vc)
        assert ((got_q - turned[:, :hq]).abs() <= bound[:, :hq])[live].all(), (tile, m)
        assert got[0][:, hq:].isnan().all()  # key and value columns go to the caches only
        at = (seq[live].long(), pos[live].long())
        assert ((kc[at[0], :, at[1]] - turned[live, hq : hq + hkv]).abs() <= bound[live, hq : hq + hkv]).all(), (tile, m)
        assert ((vc[at[0], :, at[1]] - z[live, hq + hkv :]).abs() <= err[live, hq + hkv :] + 1e-30).all(), (tile, m)
        kc[at[0], :, at[1]] = vc[at[0], :, at[1]] = float("nan")
        assert kc.isnan().all() and vc.isnan().all()


@pytest.mark.parametrize("rows", [18, 41, 100, 143, 190, 250, 300, 450, 590, 639, 720, 900, 1100, 1180])
def test_prompt_and_step(rows):
    shape = synth.StageShape("bf16", 1, 256, 16, 16, 128, 256, 0)
    first = rows // 2 + 1
    run(shape, [first, rows - first - 5, 5], 1, rows)


@pytest.mark.parametrize("rows", [60, 333])
def test_heads_of_64_columns_grouped(rows):
    run(synth.StageShape("bf16", 1, 256, 12, 3, 64, 256, 0), [rows - 9, 9], 1, rows)
