"""Infinite and NaN keys and values in fp32 attention: they reach the rows that see their key, as they did
when keys were visited one after the other, and no others."""
import pytest
import torch

import synth
from helpers import make_gpu, to_dev

pytestmark = pytest.mark.gpu

SHAPES = {hd: synth.StageShape("f32", 1, 256, 4, 2, hd, 512, 0) for hd in (64, 128)}


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("poison", [float("nan"), float("inf")])
@pytest.mark.parametrize("lengths,at", [([100], 99), ([100], 70), ([33, 130], 63), ([200], 128), ([20], 1)])
def test_prompt_rows_before_a_poisoned_token_are_what_they_are_without_it(hd, poison, lengths, at):
    T = sum(lengths)
    first = T - lengths[-1]  # the poisoned sequence is the last one
    gpu = make_gpu(SHAPES[hd], 3, 0, 1, len(lengths), max(lengths), T)
    x = to_dev(SHAPES[hd], synth.hidden_states(SHAPES[hd], 4, T))
    clean = gpu.prefill(x, lengths).clone()
    x[first + at, 5] = poison  # its normalised row is NaN, and so are its keys and values
    got = gpu.prefill(x, lengths)
    # the poisoned tile adds in another order: sums of at most 200 terms in 24 bits
    assert torch.allclose(got[: first + at], clean[: first + at], rtol=0, atol=1e-5 * float(clean.abs().max()))
    assert torch.isnan(got[first + at :]).all()  # every later row of the sequence sees the key
    gpu.close()


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("ctx,at", [(1, 0), (50, 0), (50, 7), (50, 49), (50, 20), (1000, 0), (1000, 131), (1000, 999), (1000, 500)])
def test_generation_step_over_a_poisoned_cache(hd, ctx, at):
    from paper_2502_09922_amd import binding as b

    shape = SHAPES[hd]
    gpu = make_gpu(shape, 5, 0, 1, 1, ctx + 8, ctx)
    gpu.prefill(to_dev(shape, synth.hidden_states(shape, 6, ctx)), [ctx])
    x = to_dev(shape, synth.hidden_states(shape, 7, 1))

    def attention():
        gpu.seq_lens.fill_(ctx)
        gpu.decode(x, 1, ctx)
        return gpu.workspace_region(b.LS_WS_ATTN, 1)[0].clone().view(2, 2, hd)  # kv head, its query heads

    clean = attention()
    k, v = (t.view(torch.float32).view(2, ctx + 8, hd) for t in (gpu.k, gpu.v))
    old = v[1, at, 3].clone()
    v[1, at, 3] = float("inf")  # weight times an infinite value: this dimension of the group's two heads
    got = attention()
    want = clean.clone()
    want[1, :, 3] = float("inf")
    assert torch.equal(got, want), (got[1, :, 3], (got != want).sum())
    v[1, at, 3] = old
    k[0, at, 2] = float("nan")  # a NaN score makes the softmax NaN
    got = attention()
    assert torch.isnan(got[0]).all() and torch.equal(got[1], clean[1])
    gpu.close()
