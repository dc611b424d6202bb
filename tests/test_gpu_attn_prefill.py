"""bf16 prompt attention alone, from the rotated queries and the caches that a pass leaves: prompts that end around the edges of
key tiles (32 and 64) and query tiles (128), few and many of them (tiles of 64 or 32 keys), and scores whose maximum keeps
growing by more, and by less, than what a rescale waits for."""
import pytest

import synth

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 159, 160, 161, 191, 192, 193]


@pytest.mark.parametrize("scale", [0.02, 0.3])
@pytest.mark.parametrize("hq,hkv,hd,lengths", [(32, 32, 128, EDGES), (32, 8, 128, EDGES), (4, 4, 128, EDGES), (4, 2, 64, EDGES), (64, 8, 128, [300, 257, 1030]),
                                               (8, 8, 128, [1030, 257])])
def test_against_float32(hq, hkv, hd, lengths, scale):
    import torch

    from paper_2502_09922_amd import Stage, binding as b

    shape = synth.StageShape("bf16", 2, 256, hq, hkv, hd, 256, 0)
    top = max(lengths) + 3
    st = Stage(shape, 0, 1, len(lengths), top, sum(lengths))
    g = torch.Generator(device="cuda").manual_seed(hq + hd)
    st.block_view(0).view(torch.bfloat16).normal_(0, scale, generator=g)
    off, nb = b.C.c_size_t(), b.C.c_size_t()
    b.check(b.lib.ls_block_tensor(b.C.byref(st.cfg), 0, 0, b.C.byref(off), b.C.byref(nb)))
    st.block_view(0)[off.value : off.value + nb.value].view(torch.bfloat16).fill_(1.0)
    st.adopt_block(0)
    st.k.view(torch.bfloat16).fill_(float("nan"))  # what lies behind a prompt is nobody's
    st.v.view(torch.bfloat16).fill_(float("nan"))
    st.prefill(torch.randn(sum(lengths), 256, device="cuda", generator=g).bfloat16(), lengths)
    q = st.workspace_region(b.LS_WS_QKV, sum(lengths))[:, : hq * hd].float().view(-1, hq, hd)
    got = st.workspace_region(b.LS_WS_ATTN, sum(lengths)).float().view(-1, hq, hd)
    kc, vc = (t.view(torch.bfloat16).view(len(lengths), hkv, top, hd) for t in (st.k, st.v))
    row, worst = 0, 0.0
    for i, n in enumerate(lengths):
        k, v = (t[i, :, :n].float().repeat_interleave(hq // hkv, 0) for t in (kc, vc))
        s = torch.bmm(q[row : row + n].transpose(0, 1).contiguous(), k.transpose(1, 2).contiguous()) / hd**0.5
        s = s.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), float("-inf"))
        p = torch.softmax(s, -1)
        want, size = torch.bmm(p, v), torch.bmm(p, v.abs())
        # probabilities and results are rounded to 8 bits (2^-9 of each), scores carry the fp32 errors of sums of hd products
        err = (got[row : row + n].transpose(0, 1) - want).abs()
        bound = 2.0**-8 * (want.abs() + size) + 2.0**-20 * hd * s.masked_fill(s.isinf(), 0.0).abs().amax(-1, keepdim=True) * size
        assert bool((err <= bound).all()), (n, (err / bound).max().item())
        worst = max(worst, (err / bound).max().item())
        row += n
    print("worst error %.2f of the bound" % worst)
    torch.cuda.synchronize()
    st.close()
