"""Layer blocks of 8 MiB and more arrive in four pieces, and a layer starts behind the first: prompt passes and
steps that run behind such copies give the bits of a stage whose weights were resident, with blocks in any
order, with profiling on, and after the blocks were forgotten and loaded again."""
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
