"""Generation steps of small fp32 models in one launch: the same bits as the separate launches give (a timed operator keeps
them apart), whole models and stages without embedding and head, in a batch with a sequence that has no room left, and over
many steps, whose tags and places follow each other."""
import pytest

import synth
from helpers import make_gpu
from paper_2502_09922_amd import binding as b

pytestmark = pytest.mark.gpu

# hidden, query heads, kv heads, head dim, ffn, vocab, most rows in one launch: the tiny model; columns that end inside a piece and
# inside a wavefront's share; heads that share keys (8 and 16 of them: two rows, one); 128 dimensions; K of O and down cut in 2 and
# 4; a column to each workgroup; at and behind the limits of ffn values; the first that are not taken: weights of a layer, vocab,
# columns, heads, query columns
SHAPES = [(256, 4, 4, 64, 688, 512, 4), (60, 2, 1, 64, 100, 33, 4), (252, 4, 2, 64, 692, 517, 4), (256, 8, 2, 64, 904, 1024, 2), (128, 3, 3, 128, 1028, 200, 2),
          (128, 8, 1, 64, 2048, 64, 1), (64, 8, 1, 64, 1400, 64, 2), (64, 16, 16, 64, 512, 64, 1), (64, 8, 4, 128, 256, 64, 2), (64, 1, 1, 128, 16, 16, 4),
          (64, 4, 1, 64, 768, 64, 4), (64, 4, 1, 64, 772, 64, 3), (64, 2, 2, 64, 2048, 64, 1), (64, 2, 2, 64, 2052, 64, 0),
          (196, 8, 1, 64, 2048, 64, 0), (256, 2, 2, 128, 688, 1028, 0), (260, 4, 4, 64, 688, 64, 0), (64, 32, 32, 64, 500, 64, 0), (64, 16, 16, 128, 52, 64, 0)]


def small_steps():
    b.lib.ls_test_small_steps.restype = b.C.c_long
    return b.lib.ls_test_small_steps()


def step_pair(shape, lo, hi, batch, lengths, max_seq, steps, seed=3, taken=True):
    """(one launch, separate launches): the outputs of every step, then the state, of two stages with the same blocks."""
    import torch

    runs = []
    for apart in (False, True):
        torch.manual_seed(seed)
        st = make_gpu(shape, 5, lo, hi, batch, max_seq, sum(lengths))
        torch.cuda.synchronize()
        if apart:
            st.probe(b.LS_OP_ATTENTION, lo, 1)
        first, last = st.first, st.last
        rows = lambda n: (torch.randint(0, shape.vocab, (n,), dtype=torch.int32, device="cuda") if first
                          else torch.randn(n, shape.hidden, device="cuda"))
        st.prefill(rows(sum(lengths)), lengths)
        outs, before = [], small_steps()
        for t in range(steps):
            o = st.decode(rows(batch), batch, min(max(lengths) + t, max_seq - 1), want_logits=last)
            outs += [x.clone() for x in (o if last else (o,))]
        assert small_steps() - before == (steps if taken and not apart else 0)
        outs += [st.k.clone(), st.v.clone(), st.seq_lens.clone()]
        outs += [st.workspace_region(w, batch).clone() for w in (b.LS_WS_QKV, b.LS_WS_ATTN, b.LS_WS_FFN)]
        torch.cuda.synchronize()
        st.close()
        runs.append(outs)
    return runs


def same_bits(one, apart):
    import torch

    off = {i: (x.float() - y.float()).abs().max().item() for i, (x, y) in enumerate(zip(one, apart, strict=True)) if not torch.equal(x, y)}
    assert not off


@pytest.mark.parametrize("batch", [1, 2, 3, 4])
@pytest.mark.parametrize("d,hq,hkv,hd,ffn,vocab,most", SHAPES)
def test_whole_model(d, hq, hkv, hd, ffn, vocab, most, batch):
    shape = synth.StageShape("f32", 3, d, hq, hkv, hd, ffn, vocab)
    same_bits(*step_pair(shape, 0, 3, batch, [1 + (7 * i) % 40 for i in range(batch)], 64, 5, taken=batch <= most))


def test_contexts_in_chunks():
    shape = synth.StageShape("f32", 2, 64, 2, 2, 64, 128, 64)
    for keys, taken in ((637, True), (640, False)):
        same_bits(*step_pair(shape, 0, 2, 1, [keys], keys + 4, 2, taken=taken))


@pytest.mark.parametrize("batch", [1, 3])
@pytest.mark.parametrize("lo,hi", [(0, 2), (1, 2), (2, 4)])
def test_stages(lo, hi, batch):
    shape = synth.StageShape("f32", 4, 256, 4, 4, 64, 688, 512)
    same_bits(*step_pair(shape, lo, hi, batch, [31 + i for i in range(batch)], 64, 4))


def test_long_contexts_and_many_steps():
    shape = synth.StageShape("f32", 2, 128, 2, 2, 64, 256, 96)
    same_bits(*step_pair(shape, 0, 2, 2, [500, 3], 640, 100))


def test_a_sequence_without_room_holds_nobody_up():
    import torch

    shape = synth.StageShape("f32", 2, 128, 2, 2, 64, 256, 0)
    outs = []
    for apart in (False, True):
        torch.manual_seed(1)
        st = make_gpu(shape, 5, 0, 2, 2, 16, 16)
        torch.cuda.synchronize()
        if apart:
            st.probe(b.LS_OP_ATTENTION, 0, 1)
        st.prefill(torch.randn(12, 128, device="cuda"), [7, 5])
        st.seq_lens.copy_(torch.tensor([16, 5], dtype=torch.int32))
        before = small_steps()
        outs.append((st.decode(torch.randn(2, 128, device="cuda"), 2, 15)[1].clone(), st.k.clone(), st.v.clone(), st.seq_lens.clone()))
        assert small_steps() - before == (0 if apart else 1)
        torch.cuda.synchronize()
        st.close()
    same_bits(*outs)
    assert outs[0][-1].tolist() == [16, 6]


def test_replayed_from_a_graph():
    import torch

    shape = synth.StageShape("f32", 2, 256, 4, 4, 64, 688, 512)
    st = make_gpu(shape, 5, 0, 2, 1, 64, 32)
    tok = torch.randint(0, 512, (1,), dtype=torch.int32, device="cuda")
    st.prefill(torch.randint(0, 512, (20,), dtype=torch.int32, device="cuda"), [20])
    torch.cuda.synchronize()
    out = torch.zeros(1, dtype=torch.int32, device="cuda")
    eager = []
    for t in range(4):
        st.decode(tok, 1, 40, out=out)
        eager.append(int(out[0]))
    st.seq_lens.fill_(20)
    torch.cuda.synchronize()
    g, side, before = torch.cuda.CUDAGraph(), torch.cuda.Stream(), small_steps()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=side):
        st.decode(tok, 1, 40, out=out, stream=side)
    assert small_steps() == before + 1
    got = []
    for t in range(4):
        g.replay()
        torch.cuda.synchronize()
        got.append(int(out[0]))
    assert got == eager and int(st.seq_lens[0]) == 24
    st.close()
