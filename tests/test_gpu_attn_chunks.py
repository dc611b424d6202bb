"""Attention at the sizes where it changes form: generation steps whose contexts are cut into chunks
that are workgroups of their own (few sequences x kv heads; contexts at and around the shortest
chunk of 128 keys and the shortest context of 640, ragged), fp32 generation steps, and the fp32 prompt
kernel (64-row query tiles, 32-key tiles, head_dim 64 and 128, grouped queries).  Against the oracle."""
import pytest

import synth
from helpers import check_close, check_delta, make_gpu, make_oracle, to_dev, to_host
from oracle.stage_oracle import decode_values

pytestmark = pytest.mark.gpu


def run(shape, lengths, steps, seed, max_ctx_of):
    B, longest, T = len(lengths), max(lengths), sum(lengths)
    gpu = make_gpu(shape, seed, 0, 1, B, longest + steps, T)
    ora = make_oracle(shape, seed, 0, 1, B, longest + steps)
    x = synth.hidden_states(shape, seed + 1, T)
    got, want = to_host(gpu.prefill(to_dev(shape, x), lengths)), ora.prefill(x, lengths)
    check_close(got, want, shape.dtype, "prompt")
    check_delta(got, want, decode_values(x), shape.dtype, "prompt")
    for t in range(steps):
        xs = synth.hidden_states(shape, seed + 2 + t, B)
        got, want = to_host(gpu.decode(to_dev(shape, xs), B, max_ctx_of(longest + t))), ora.decode(xs)
        check_close(got, want, shape.dtype, "step %d" % t)
    gpu.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("heads", [(2, 2, 128), (4, 2, 64), (4, 1, 64)])
@pytest.mark.parametrize("lengths", [[1], [127], [128], [129], [639], [640, 3, 130], [1101], [1, 33, 64, 65, 95, 97]])
def test_contexts_at_chunk_and_tile_edges(dtype, heads, lengths):
    hq, hkv, hd = heads
    shape = synth.StageShape(dtype, 1, 256, hq, hkv, hd, 512, 0)
    run(shape, lengths, 2, sum(lengths), lambda ctx: ctx)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_a_context_longer_than_the_caller_names(dtype):
    """max_ctx sizes the chunks; a sequence that is longer all the same is read to its end."""
    shape = synth.StageShape(dtype, 1, 256, 2, 2, 64, 512, 0)
    run(shape, [1000, 40], 1, 9, lambda ctx: 700)
