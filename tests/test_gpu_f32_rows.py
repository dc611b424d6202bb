"""Few fp32 rows through the projections that take the rows' norm along and add to the residual rows themselves: widths
that end inside a 256-column piece, the widest that are taken and the first that is not, every row count up
to nine, ragged outputs, a stage's hidden rows and a whole model's logits."""
import pytest

import synth
from helpers import TOL, check_close, make_gpu, make_oracle, to_dev, to_host
from paper_2502_09922_amd import binding as b
from test_gpu_parity import run_full_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", range(1, 10))
@pytest.mark.parametrize("d,ffn,vocab", [(60, 100, 33), (256, 688, 512), (260, 692, 517), (1024, 340, 301), (1028, 256, 64)])
def test_whole_model(d, ffn, vocab, batch):
    shape = synth.StageShape("f32", 2, d, 2, 1, 64, ffn, vocab)
    errs, agree = run_full_model(shape, d + batch, [1 + (3 * i) % 7 for i in range(batch)], 2)
    assert max(errs) <= TOL["f32"], errs
    assert all(adj == n for _, adj, n in agree), agree


@pytest.mark.parametrize("d", [256, 500, 1024])
@pytest.mark.parametrize("batch", [1, 2, 3, 8])
def test_norm_on_its_own_gives_the_same_bits(d, batch):
    import torch

    shape = synth.StageShape("f32", 3, d, 2, 2, 64, 692, 0)
    lengths = [5 + i for i in range(batch)]
    gpu, ora = make_gpu(shape, 3, 0, 3, batch, 32, sum(lengths)), make_oracle(shape, 3, 0, 3, batch, 32)
    x = synth.hidden_states(shape, 4, sum(lengths))
    gpu.prefill(to_dev(shape, x), lengths)
    ora.prefill(x, lengths)
    xs = synth.hidden_states(shape, 5, batch)
    want, outs = ora.decode(xs), []
    for layer in (None, 0, 1, 2):  # a timed norm is a launch of its own
        gpu.probe(b.LS_OP_NONE if layer is None else b.LS_OP_NORM, layer or 0, 1)
        gpu.seq_lens.copy_(torch.tensor(lengths, dtype=torch.int32))
        outs.append(gpu.decode(to_dev(shape, xs), batch, max(lengths)).clone())
        check_close(to_host(outs[-1]), want, "f32", "norm of layer %s alone" % layer)
        assert torch.equal(outs[0], outs[-1]), layer
    gpu.close()
