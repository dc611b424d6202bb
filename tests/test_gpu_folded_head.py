"""The final norm folded into the LM head of bf16 generation steps of up to 16 rows: row counts up to the first that keeps
the norm's own launch, vocabularies that the weight-streaming GEMM takes and one that it does not, a hidden size whose
sums of squares need a second request, rows of a caller's logits buffer beside the library's own."""
import pytest

import synth
from helpers import TOL, make_gpu, to_dev
from test_gpu_parity import run_full_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [16, 1000, 1008])
@pytest.mark.parametrize("batch", [1, 3, 8, 9, 16, 17])
def test_logits_and_tokens(vocab, batch):
    shape = synth.StageShape("bf16", 1, 512, 4, 2, 128, 640, vocab)
    errs, agree = run_full_model(shape, vocab + batch, [1 + (3 * i) % 7 for i in range(batch)], 2)
    assert max(errs) <= TOL["bf16"], errs
    assert all(adj == n for _, adj, n in agree), agree


@pytest.mark.parametrize("batch", [1, 8])
def test_hidden_size_of_more_than_4096(batch):
    errs, _ = run_full_model(synth.StageShape("bf16", 1, 4608, 4, 4, 128, 512, 272), batch, [3] * batch, 1)
    assert max(errs) <= TOL["bf16"], errs


def test_same_tokens_without_a_logits_buffer():
    import torch

    shape = synth.StageShape("bf16", 2, 512, 4, 4, 128, 640, 1008)
    gpu = make_gpu(shape, 7, 0, 2, 5, 16, 20)
    gpu.prefill(to_dev(shape, synth.token_ids(8, 20, shape.vocab)), [4] * 5)
    tok = to_dev(shape, synth.token_ids(9, 5, shape.vocab))
    with_logits, _ = gpu.decode(tok, 5, 4, want_logits=True)
    gpu.seq_lens.copy_(torch.full((5,), 4, dtype=torch.int32))
    assert torch.equal(with_logits, gpu.decode(tok, 5, 4))
    gpu.close()
