"""Few fp32 rows through the projections that take the rows' norm along and add to the residual rows themselves: widths
that end inside a 256-column piece, the widest that are taken and the first that is not, every row count up
to nine, as many pieces of 256 columns as are taken and one more, heads of as many entries and more, ragged outputs, a
stage's hidden rows and a whole model's logits."""
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


@pytest.mark.parametrize("d,vocab,batch", [(256, 20000, 8), (256, 20004, 8), (384, 32001, 2), (384, 32001, 3), (768, 40, 5), (768, 40, 6)])
def test_heads_and_widths_around_what_is_taken(d, vocab, batch):
    shape = synth.StageShape("f32", 1, d, 2, 2, 64, 340, vocab)
    errs, agree = run_full_model(shape, vocab + d, [1 + (3 * i) % 7 for i in range(batch)], 1)
    assert max(errs) <= TOL["f32"], errs
    assert all(adj == n for _, adj, n in agree), agree


@pytest.mark.parametrize("d", [384, 768])
def test_eight_rows_take_no_longer_than_nine(d):
    """Nine rows go through the tiled GEMM, with norms of their own.  (A norm in each wavefront of the head, 32000 entries, 384
    columns: 8 rows 149 us, 9 rows 65; 768 columns: 159 and 91.)"""
    import torch

    gpu = make_gpu(synth.StageShape("f32", 2, d, d // 64, d // 64, 64, 1376, 32000), 1, 1, 2, 9, 64, 9)
    x = torch.randn(9, d, device="cuda")
    best = {}
    for _ in range(5):
        for rows in (8, 9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            for i in range(45):
                if i == 5:
                    a.record()
                gpu.seq_lens.fill_(20)
                gpu.decode(x[:rows], rows, 20)
            b.record()
            torch.cuda.synchronize()
            best[rows] = min(best.get(rows, 1e9), a.elapsed_time(b) / 40)
    gpu.close()
    print("8 rows %.1f us, 9 rows %.1f us" % (1e3 * best[8], 1e3 * best[9]))
    assert best[8] <= 1.2 * best[9]


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
