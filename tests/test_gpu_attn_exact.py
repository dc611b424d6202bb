"""What bf16 prompt attention must not lose: the largest probability of a row, which is 1 and exact in bf16, however the row's
maximum grows from key tile to key tile; from the rotated queries and the caches that a pass leaves."""
import pytest

import synth

pytestmark = pytest.mark.gpu


def stage_of(hq, hkv, hd, lengths, fill):
    """A one-layer stage of 256 columns; fill(wqkv) sets its projection, the other weights are small and normal."""
    import torch

    from paper_2502_09922_amd import Stage, binding as b

    shape = synth.StageShape("bf16", 2, 256, hq, hkv, hd, 256, 0)
    st = Stage(shape, 0, 1, len(lengths), max(lengths), sum(lengths))
    block = st.block_view(0)
    block.view(torch.bfloat16).normal_(0, 0.02, generator=torch.Generator(device="cuda").manual_seed(1))
    for i in (0, 1):
        off, nb = b.C.c_size_t(), b.C.c_size_t()
        b.check(b.lib.ls_block_tensor(b.C.byref(st.cfg), 0, i, b.C.byref(off), b.C.byref(nb)))
        t = block[off.value : off.value + nb.value].view(torch.bfloat16)
        t.fill_(1.0) if i == 0 else fill(t.view(-1, 256))
    st.adopt_block(0)
    return st


def attention(st, hq, hkv, hd, x, lengths):
    """(attention output, scores in float64, masked, values) of every sequence, heads first."""
    import torch

    from paper_2502_09922_amd import binding as b

    st.prefill(x, lengths)
    q = st.workspace_region(b.LS_WS_QKV, sum(lengths))[:, : hq * hd].double().view(-1, hq, hd)
    got = st.workspace_region(b.LS_WS_ATTN, sum(lengths)).double().view(-1, hq, hd)
    kc, vc = (t.view(torch.bfloat16).view(len(lengths), hkv, max(lengths), hd) for t in (st.k, st.v))
    row = 0
    for i, n in enumerate(lengths):
        k, v = (t[i, :, :n].double().repeat_interleave(hq // hkv, 0) for t in (kc, vc))
        s = torch.bmm(q[row : row + n].transpose(0, 1).contiguous(), k.transpose(1, 2).contiguous()) / hd**0.5
        yield got[row : row + n].transpose(0, 1), s.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), float("-inf")), v
        row += n


@pytest.mark.parametrize("hq,hkv,hd,lengths", [(8, 8, 128, [311, 70]), (32, 8, 128, [193, 130, 97] * 8), (8, 2, 64, [311, 70])])
def test_the_largest_probability_is_exact(hq, hkv, hd, lengths):
    import torch

    g = torch.Generator(device="cuda").manual_seed(hq + hd)
    st = stage_of(hq, hkv, hd, lengths, lambda w: w.normal_(0, 0.2, generator=g))
    x = torch.randn(sum(lengths), 256, device="cuda", generator=g).bfloat16()
    seen = 0
    for got, s, v in attention(st, hq, hkv, hd, x, lengths):
        p = torch.softmax(s, -1)
        want = torch.bmm(p, v)
        top = p.argmax(-1, keepdim=True)
        rest = torch.bmm(p.scatter(-1, top, 0.0), v.abs()) + (1.0 - p.gather(-1, top)) * want.abs()
        # half a last bit of the result.  All else is lost on the other keys: their probabilities' last bits, and the fp32
        # errors of scores (sums of hd products), which move weight between the keys.  1e-5: fp32 factors and quotient
        size = s.masked_fill(s.isinf(), 0.0).abs().amax(-1, keepdim=True)
        bound = (2.0**-8 + 1e-5) * want.abs() + (2.0**-8 + 2.0**-20 * hd * size) * rest
        assert bool(((got - want).abs() <= bound).all()), ((got - want).abs() / bound).max().item()
        seen += int((p.amax(-1) > 0.999).sum())
    assert seen > 100  # rows that are nothing but their largest probability
    torch.cuda.synchronize()
    st.close()


@pytest.mark.parametrize("hq,hkv,lengths", [(32, 32, [100] * 20), (32, 8, [97, 40] * 24), (4, 4, [100, 200])])
@pytest.mark.parametrize("first", [31, 32, 33, 64])
def test_first_keys_whose_scores_overflow_count_nothing(hq, hkv, lengths, first):
    """The first keys of a prompt score -inf in all later rows: a whole key tile of them, more and less."""
    import torch

    hd = 128

    def fill(w):
        # the slowest pair of each head, which positions hardly turn, multiplies column 0 (keys) and column 1 (queries); the
        # rest knows neither
        w.normal_(0, 0.05, generator=torch.Generator(device="cuda").manual_seed(7))
        w[:, :2] = 0.0
        qk = w[: (hq + hkv) * hd].view(-1, hd, 256)
        qk[:, hd - 2 :] = 0.0
        qk[:hq, hd - 2, 1] = 1e20
        qk[hq:, hd - 2, 0] = -1e20

    lengths = [max(n, first + 5) for n in lengths]
    st = stage_of(hq, hkv, hd, lengths, fill)
    x = torch.randn(sum(lengths), 256, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).bfloat16()
    x[:, 0], x[:, 1] = 0.0, 1.0
    row = 0
    for n in lengths:
        x[row : row + first, 0], x[row : row + first, 1] = 1.0, 0.0
        row += n
    for (got, s, v), n in zip(attention(st, hq, hkv, hd, x, lengths), lengths):
        assert bool((s[:, first:, :first].masked_fill(s[:, first:, :first].isnan(), 0) < -1e38).all())
        s[:, first:, :first] = float("-inf")
        p = torch.softmax(s, -1)
        want, size = torch.bmm(p, v), torch.bmm(p, v.abs())
        # probabilities and results are rounded to 8 bits; scores, none beyond 100 here, carry the errors of sums of hd products
        bound = 2.0**-7 * (want.abs() + size) + 2.0**-20 * hd * 100 * size
        assert bool(((got - want).abs() <= bound).all())
    torch.cuda.synchronize()
    st.close()
