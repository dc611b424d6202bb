"""The tiled GEMM and the one-pass row kernel (gemm_tiled.*) at the sizes where they can go wrong:
row counts at the edges of their tiles (32, 64, 96, 128, 160, 256 rows, one more, one less), widths that
end inside a tile, fp32 K with half a k-step at its end (688 = 21.5 x 32), K split several ways,
generation steps of more than 64 rows, heads of 32 columns (no MFMA attention), a width the row
kernel does not take.  Prompt pass and generation steps through the C ABI against the oracle."""
import numpy as np
import pytest

import synth
from helpers import check_close, check_delta, make_gpu, make_oracle, to_dev, to_host
from oracle.stage_oracle import decode_values

pytestmark = pytest.mark.gpu

S = synth.StageShape
SHAPES = {
    # dtype, layers, hidden, q heads, kv heads, head dim, ffn, vocab
    "f32": S("f32", 2, 256, 4, 2, 64, 688, 0),
    "f32_ragged": S("f32", 1, 208, 4, 4, 32, 176, 0),  # K = 208, 128, 176: half k-steps, hidden not a tile's width
    "bf16": S("bf16", 2, 512, 4, 2, 128, 1408, 0),
    "bf16_ragged": S("bf16", 1, 416, 3, 1, 64, 352, 0),  # K = 416 and 352: half k-steps
    "bf16_hd32": S("bf16", 1, 256, 8, 8, 32, 512, 0),
    "bf16_wide": S("bf16", 1, 8224, 2, 1, 128, 256, 0),  # wider than the row kernel: separate passes
}


def run(shape, lengths, steps, seed):
    B, longest, T = len(lengths), max(lengths), sum(lengths)
    gpu = make_gpu(shape, seed, 0, shape.n_layers_total, B, longest + steps, T)
    ora = make_oracle(shape, seed, 0, shape.n_layers_total, B, longest + steps)
    x = synth.hidden_states(shape, seed + 1, T)
    got, want = to_host(gpu.prefill(to_dev(shape, x), lengths)), ora.prefill(x, lengths)
    tag = "%s T%d" % (shape.dtype, T)
    check_close(got, want, shape.dtype, tag + " prompt")
    check_delta(got, want, decode_values(x), shape.dtype, tag + " prompt")
    for t in range(steps):
        xs = synth.hidden_states(shape, seed + 2 + t, B)
        got, want = to_host(gpu.decode(to_dev(shape, xs), B, longest + t)), ora.decode(xs)
        check_close(got, want, shape.dtype, tag + " step %d" % t)
    gpu.close()


@pytest.mark.parametrize("rows", [1, 17, 32, 33, 64, 65, 96, 97, 128, 129, 160, 161, 255, 257, 320, 513])
@pytest.mark.parametrize("name", ["f32", "bf16"])
def test_prompt_rows_at_tile_edges(name, rows):
    run(SHAPES[name], [rows - rows // 3, rows // 3] if rows >= 3 else [rows], 1, rows)


@pytest.mark.parametrize("name", ["f32_ragged", "bf16_ragged", "bf16_hd32", "bf16_wide"])
@pytest.mark.parametrize("rows", [40, 100])
def test_shapes_that_end_inside_a_tile_or_take_the_separate_passes(name, rows):
    run(SHAPES[name], [rows - 7, 7], 2, rows)


@pytest.mark.parametrize("name", ["f32", "bf16"])
@pytest.mark.parametrize("batch", [65, 100, 129])
def test_generation_steps_of_more_than_64_rows(name, batch):
    run(SHAPES[name], [1 + (5 * i) % 9 for i in range(batch)], 2, batch)


def test_head_and_embedding_in_fp32_and_of_more_than_64_rows():
    from helpers import TOL
    from test_gpu_parity import run_full_model

    for shape, lengths in ((S("f32", 2, 256, 4, 4, 64, 688, 1000), [33, 5, 1]),
                           (S("bf16", 2, 256, 4, 4, 64, 704, 1008), [2 + i % 3 for i in range(70)])):
        errs, agree = run_full_model(shape, 3, lengths, 2)
        assert max(errs) <= TOL[shape.dtype], (shape, errs)
        assert sum(a[1] for a in agree) >= 0.99 * sum(a[2] for a in agree)


@pytest.mark.parametrize("name,batch", [("f32", 3), ("bf16", 66)])
def test_input_and_output_buffers_at_odd_addresses(name, batch):
    import torch

    shape = SHAPES[name]
    gpu = make_gpu(shape, 5, 0, 2, batch, 8, 2 * batch)
    x = to_dev(shape, synth.hidden_states(shape, 6, 2 * batch))

    def odd(t):  # a copy one element past an aligned address
        room = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        room[1:] = t.reshape(-1)
        return room[1:].view(t.shape)

    def both(inp, out):
        prompt = gpu.prefill(inp, [2] * batch)
        return prompt, gpu.decode(odd(x[:batch]), batch, 2, out=out).clone()

    want = both(x, None)
    got = both(odd(x), odd(torch.zeros_like(x[:batch])))
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])
    gpu.close()


def test_fp32_infinities_pass_through_the_split_products():
    """Large fp32 tiles are multiplied as bf16 parts, which an infinity does not have: a k-step that holds one is
    multiplied in fp32, and every other column of the row stays what it is."""
    import torch

    shape = S("f32", 1, 512, 4, 4, 64, 512, 0)
    lengths = [460] * 5
    rows = sum(lengths)
    from paper_2502_09922_amd import binding as b
    import ctypes as C

    plan = (C.c_int * 3)()
    fn = b.lib.ls_test_tiled_plan
    fn.argtypes = [C.c_uint32] + [C.c_int] * 5 + [C.c_size_t, C.POINTER(C.c_int * 3)]
    assert fn(0, 0, rows, 512, 512, 1, 8 * rows * 512 * 4, C.byref(plan))  # the down projection of this call
    assert plan[0] * plan[1] >= 96 * 128, list(plan)  # goes by the parts
    gpu = make_gpu(shape, 11, 0, 1, 5, 512, rows)
    view = gpu.block_view(0)

    off, nb = C.c_size_t(), C.c_size_t()
    b.check(b.lib.ls_block_tensor(C.byref(gpu.cfg), 0, 5, C.byref(off), C.byref(nb)))  # w_down [hidden, ffn]
    wd = view[off.value : off.value + nb.value].view(torch.float32).view(512, 512)
    x = to_dev(shape, synth.hidden_states(shape, 12, rows))
    clean = gpu.prefill(x, lengths).clone()
    h = gpu.workspace_region(b.LS_WS_FFN, rows).clone()
    wd[7, 100] = float("inf")
    got = gpu.prefill(x, lengths)
    others = torch.arange(512, device="cuda") != 7
    scale = clean.abs().max()
    assert ((got - clean)[:, others].abs() <= 1e-5 * scale).all()
    want = torch.where(h[:, 100] > 0, float("inf"), -float("inf"))
    assert torch.equal(got[:, 7], want)
    gpu.close()


@pytest.mark.parametrize("dtype,rows,width", [("bf16", 2049, 1024), ("bf16", 2300, 1056), ("bf16", 2300, 1040),
                                              ("bf16", 2300, 8192), ("f32", 2300, 8192)])
def test_many_rows_against_the_same_rows_a_few_at_a_time(dtype, rows, width):
    """256 x 256 tiles whose epilogue stores the stage's output rows (widths that are a multiple of 32 or, 1040, not),
    and rows whose partial tiles would not fit the scratch (8192 columns: 75 MB), against shorter calls."""
    shape = S(dtype, 1, width, 4, 4, 128, 1024, 0)
    gpu = make_gpu(shape, 21, 0, 1, 24, 128, rows)
    lengths = [100] * (rows // 100) + ([rows % 100] if rows % 100 else [])
    x = to_dev(shape, synth.hidden_states(shape, 22, rows))
    whole = gpu.prefill(x, lengths).clone()
    parts, r = [], 0
    for n in lengths:
        parts.append(gpu.prefill(x[r : r + n].contiguous(), [n]).clone())
        r += n
    got, want = to_host(whole), np.concatenate([to_host(p) for p in parts])
    # both paths round the same places (bf16: to 8 bits) and add in another order: at most a few roundings apart
    assert np.linalg.norm(got - want) <= (5e-3 if dtype == "bf16" else 1e-5) * np.linalg.norm(want)
    gpu.close()
