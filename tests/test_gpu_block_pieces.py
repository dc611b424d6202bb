"""Layer blocks of 8 MiB and more arrive in four pieces, and a layer starts behind the first: prompt passes and
steps that run behind such copies give the bits of a stage whose weights were resident, with blocks in any
order, with profiling on, and after the blocks were forgotten and loaded again.  A head block arrives in two."""
import time

import pytest

import synth
from helpers import make_gpu, packed_blocks, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [(0, 1), (1, 0)])
@pytest.mark.parametrize("rows", [9, 200])
def test_a_pass_behind_pieces_equals_a_pass_on_resident_weights(order, rows):
    import torch

    shape = synth.StageShape("bf16", 2, 1024, 8, 8, 128, 2816, 0)
    st = make_gpu(shape, 3, 0, 2, 1, 256, 256)
    assert st.slab.numel() >= 2 * (8 << 20)
    x = to_dev(shape, synth.hidden_states(shape, 4, rows))
    want = st.prefill(x, [rows]).clone()
    step = st.decode(x[:1], 1, rows).clone()
    host = {l: st.stage_host_block(l, buf) for l, buf in packed_blocks(st, 3).items()}
    copies = torch.cuda.Stream()
    for profiling in (False, True, False):
        torch.cuda.synchronize()
        st.set_profiling(profiling)
        st.reset_blocks()
        st.slab.zero_()
        copies.wait_stream(torch.cuda.current_stream())
        for l in order:
            st.load_block(l, host[l], copies)
        got = st.prefill(x, [rows])
        assert torch.equal(got, want)
        assert torch.equal(st.decode(x[:1], 1, rows), step)
    st.close()


def test_a_step_waits_for_the_lm_head_only_in_front_of_it():
    """A step of few rows applies the final norm's gain in its last down projection; the LM head behind the gain, 512 MB, is
    still on its way when that is done.  Same bits as with resident weights."""
    import torch
    from paper_2502_09922_amd import LsError, binding

    shape = synth.StageShape("bf16", 2, 1024, 8, 8, 128, 2816, 262144)
    st = binding.Stage(shape, 1, 2, 2, 16, 16)
    gen = torch.Generator(device="cuda").manual_seed(5)
    host = {}
    for layer in st.block_ids():
        view = st.block_view(layer)
        view.view(torch.bfloat16).normal_(0, 0.02, generator=gen)
        host[layer] = torch.empty(view.numel(), dtype=torch.uint8, pin_memory=True)
        host[layer].copy_(view)
        st.adopt_block(layer)
    x = torch.randn(2, 1024, generator=gen, device="cuda").to(torch.bfloat16)
    _, want = st.decode(x, 2, 0, want_logits=True)
    overlapped = False
    for attempt in range(8):  # streams share four hardware queues: one that is the step's own holds the step back by itself
        copies = torch.cuda.Stream()
        torch.cuda.synchronize()
        st.reset_blocks()
        st.slab.zero_()
        st.seq_lens.zero_()
        st.probe(binding.LS_OP_GEMM_DOWN, 1, 1)
        torch.cuda.synchronize()
        for layer in (2, 1) if attempt == 7 else (1, 2):
            st.load_block(layer, host[layer], copies)
        _, got = st.decode(x, 2, 0, want_logits=True)
        time.sleep(0.004)  # the layer arrives in 0.4 ms, the head takes 9
        try:
            st.probe_times()  # an error as long as the projection is not done
            overlapped |= not copies.query()
        except LsError:
            binding.lib.hipGetLastError()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    assert overlapped
    st.close()
