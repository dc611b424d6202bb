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
