"""The first residual add of a stage that is given hidden rows.  Many bf16 rows are added to where they lie, others are widened to
fp32 first; a buffer that no eight-byte load may read always takes the second way, and both give the same bits."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,hq,hkv,hd,lengths", [
    (1028, 4, 2, 64, [65]),  # columns that end inside a tile and a group of 32
    (260, 4, 4, 64, [129, 128, 1]),
    (1024, 8, 8, 128, [4097]),
    (4096, 32, 8, 128, [1500, 1, 2600]),
    (256, 2, 2, 128, [33, 32]),
])
@pytest.mark.parametrize("layers", [1, 2])
def test_same_bits_wherever_the_rows_lie(hidden, hq, hkv, hd, lengths, layers):
    import torch

    from paper_2502_09922_amd import Stage

    shape = synth.StageShape("bf16", 4, hidden, hq, hkv, hd, 512, 0)
    rows = sum(lengths)
    st = Stage(shape, 1, 1 + layers, len(lengths), max(lengths) + 4, rows)
    g = torch.Generator(device="cuda").manual_seed(hidden)
    for i in st.block_ids():
        st.block_view(i).view(torch.bfloat16).normal_(0, 0.05, generator=g)
        st.adopt_block(i)
    flat = torch.empty(rows * hidden + 8, device="cuda", dtype=torch.bfloat16)
    values = torch.randn(rows, hidden, device="cuda", generator=g).bfloat16()
    got = []
    for shift in (0, 4, 1, 2):  # the last two are no multiple of eight bytes
        x = flat[shift : shift + rows * hidden].view(rows, hidden)
        x.copy_(values)
        # what an earlier call left must not be what the rows are added to
        st.prefill(torch.randn(rows, hidden, device="cuda", generator=g).bfloat16(), lengths)
        got.append(st.prefill(x, lengths).clone())
    torch.cuda.synchronize()
    assert bool(got[0].isfinite().all())
    for other in got[1:]:
        assert torch.equal(got[0], other)
    st.close()


def test_rows_in_host_memory_are_read_once():
    """By the first row kernel: the O projection takes as long as with rows in device memory (over the host link their 32 MB alone
    would take four times that)."""
    import torch

    from paper_2502_09922_amd import Stage, binding as b

    shape = synth.StageShape("bf16", 4, 4096, 32, 8, 128, 512, 0)
    lengths = [1500, 1, 2595]
    st = Stage(shape, 1, 2, len(lengths), max(lengths) + 4, sum(lengths))
    for i in st.block_ids():
        st.block_view(i).view(torch.bfloat16).normal_(0, 0.05, generator=torch.Generator(device="cuda").manual_seed(1))
        st.adopt_block(i)
    rows = torch.randn(sum(lengths), 4096, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2)).bfloat16()
    pinned = torch.empty(rows.shape, dtype=rows.dtype, pin_memory=True)
    pinned.copy_(rows)
    out, time = [], []
    for x in (rows, pinned):
        st.prefill(x, lengths)
        st.probe(b.LS_OP_GEMM_O, 1, 0)
        for _ in range(5):
            out.append(st.prefill(x, lengths).clone())
        torch.cuda.synchronize()
        time.append(min(st.probe_times()))
        st.probe(b.LS_OP_NONE)
    print("O projection %.3f ms, rows in host memory %.3f ms" % tuple(time))
    assert all(torch.equal(o, out[0]) for o in out)
    assert time[1] < 2 * time[0]
    st.close()
