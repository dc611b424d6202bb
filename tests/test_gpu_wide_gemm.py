"""The weight-streaming GEMM for 17..64 rows (gemm_skinny_wide.hip) where it still serves: stages of hidden sizes
above 8192, which the one-pass row kernel does not take (prompts, and generation steps with the norms folded
in, with and without K cut across workgroups), and logits of 17..64 rows at an address that is not
16-byte aligned."""
import ctypes as C

import pytest

import synth
from helpers import TOL, check_close, check_delta, make_gpu, make_oracle, to_dev, to_host
from oracle.stage_oracle import decode_values

pytestmark = pytest.mark.gpu

# hidden, qkv columns, attention columns and ffn are multiples of 128 from 512 on: all four projections
WIDE = synth.StageShape("bf16", 2, 8320, 4, 1, 128, 512, 0)


@pytest.mark.parametrize("batch", [17, 32, 33, 64])
def test_layers_wider_than_the_row_kernel(batch):
    gpu = make_gpu(WIDE, 7, 0, 2, batch, 8, batch)
    ora = make_oracle(WIDE, 7, 0, 2, batch, 8)
    x = synth.hidden_states(WIDE, 8, batch)
    got, want = to_host(gpu.prefill(to_dev(WIDE, x), [1] * batch)), ora.prefill(x, [1] * batch)
    check_close(got, want, "bf16", "prompt")
    check_delta(got, want, decode_values(x), "bf16", "prompt")
    for t in range(2):
        xs = synth.hidden_states(WIDE, 9 + t, batch)
        want = ora.decode(xs)
        gpu.seq_lens.fill_(1 + t)
        got = to_host(gpu.decode(to_dev(WIDE, xs), batch, 1 + t))
        check_close(got, want, "bf16", "step %d" % t)
        gpu.seq_lens.fill_(1 + t)
        assert (to_host(gpu.decode(to_dev(WIDE, xs), batch, 1 + t, static=True)) == got).all()
    gpu.close()


@pytest.mark.parametrize("batch", [17, 32, 64])
def test_logits_at_an_odd_address(batch):
    import torch
    from paper_2502_09922_amd import binding as b

    shape = synth.StageShape("bf16", 1, 512, 4, 2, 128, 1408, 1024)
    gpu = make_gpu(shape, 5, 0, 1, batch, 8, batch)
    ora = make_oracle(shape, 5, 0, 1, batch, 8)
    tok = synth.token_ids(6, batch, shape.vocab)
    ora.prefill(tok, [1] * batch)
    gpu.prefill(to_dev(shape, tok), [1] * batch)
    tok = synth.token_ids(7, batch, shape.vocab)
    want = ora.decode(tok)[1]
    feed, nxt = to_dev(shape, tok), torch.empty(batch, dtype=torch.int32, device="cuda")
    room = torch.full((batch * shape.vocab + 2,), 7.0, device="cuda")
    b.check(b.lib.ls_stage_decode(gpu.handle, feed.data_ptr(), batch, 1, C.byref(gpu.kv), nxt.data_ptr(),
                                  room.data_ptr() + 4, gpu._stream_ptr(None)))
    torch.cuda.synchronize()
    assert room[0] == 7.0 and room[-1] == 7.0
    got = room[1:-1].view(batch, shape.vocab)
    assert check_close(to_host(got), want, "bf16", "logits")["rel_l2"] <= TOL["bf16"]
    assert torch.equal(nxt.long(), got.argmax(1))
    gpu.close()
