"""The sequence bounds of a prompt pass: written in stream order on the current stream (more of them than one kernel
carries), copied where the pass runs on another stream or reads rows in pinned host memory; passes one behind the other with nothing
waited for between them."""
import ctypes as C
import time

import numpy as np
import pytest

import synth
from helpers import make_gpu, to_dev
from paper_2502_09922_amd import LsError, binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 1000])
def test_write_ints(n):
    import torch

    host = np.arange(7, 7 + max(n, 1), dtype=np.int32)
    dev = torch.full((n + 2,), -1, dtype=torch.int32, device="cuda")
    binding.check(binding.lib.ls_write_ints(dev.data_ptr(), host.ctypes.data_as(C.POINTER(C.c_int32)), n, None))
    host[:] = 0  # the call has taken the values
    assert dev.cpu().tolist() == list(range(7, 7 + n)) + [-1, -1]
    with pytest.raises(LsError):
        binding.check(binding.lib.ls_write_ints(dev.data_ptr(), host.ctypes.data_as(C.POINTER(C.c_int32)), -1, None))


def test_passes_without_a_wait_between_them():
    import torch

    shape = synth.StageShape("bf16", 1, 256, 2, 2, 128, 256, 0)
    gpu = make_gpu(shape, 3, 0, 1, 300, 8, 1200)
    side = torch.cuda.Stream()
    gpu.prefill(to_dev(shape, synth.hidden_states(shape, 9, 3)), [3])  # behind the load
    lens = [[1 + (i * k) % 4 for i in range(300)] for k in (1, 2, 3)] + [[4, 2, 1], [8]]
    xs = [to_dev(shape, synth.hidden_states(shape, 4 + i, sum(n))) for i, n in enumerate(lens)]
    torch.cuda.synchronize()
    outs = [gpu.prefill(x, n) for x, n in zip(xs, lens)]
    torch.cuda.synchronize()
    for x, n, out in zip(xs, lens, outs):
        other = gpu.prefill(x, n, stream=side)
        torch.cuda.synchronize()
        assert torch.equal(out, other)
        with torch.cuda.stream(side):
            same = gpu.prefill(x, n, stream=side)
        torch.cuda.synchronize()
        assert torch.equal(out, same)
        assert gpu.seq_lens[: len(n)].cpu().tolist() == n
    gpu.close()


def test_rows_in_pinned_host_memory():
    import torch

    shape = synth.StageShape("bf16", 1, 256, 2, 2, 128, 256, 0)
    gpu = make_gpu(shape, 3, 0, 1, 4, 64, 256)
    x = to_dev(shape, synth.hidden_states(shape, 5, 64))
    for lens in ([64], [3, 40, 21]):
        want = gpu.prefill(x, lens).clone()
        host = torch.empty(x.shape, dtype=x.dtype, pin_memory=True)
        host.copy_(x)
        assert torch.equal(gpu.prefill(host, lens), want)
        assert torch.equal(gpu.prefill(host, lens), want)
        assert torch.equal(gpu.prefill(x, lens), want)
    gpu.close()


def test_the_host_does_not_wait_for_arriving_blocks():
    """Load and run, twice: all of it is enqueued while the first blocks are still on their way (a copy of the bounds from
    pageable memory waited for the pass before, 9 ms)."""
    import torch

    shape = synth.StageShape("bf16", 2, 4096, 32, 32, 128, 11008, 0)
    st = binding.Stage(shape, 0, 2, 1, 64, 64)
    gen = torch.Generator(device="cuda").manual_seed(5)
    host = []
    for layer in st.block_ids():
        view = st.block_view(layer)
        view.view(torch.bfloat16).normal_(0, 0.02, generator=gen)
        host.append(torch.empty(view.numel(), dtype=torch.uint8, pin_memory=True))
        host[-1].copy_(view)
        st.adopt_block(layer)
    x = torch.randn(64, 4096, generator=gen, device="cuda").to(torch.bfloat16)
    want = st.prefill(x[:40], [40]).clone()
    copies = torch.cuda.Stream()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    outs = []
    for _ in range(2):
        st.reset_blocks()
        copies.wait_stream(torch.cuda.current_stream())
        for layer, t in zip(st.block_ids(), host):
            st.load_block(layer, t, copies)
        outs.append(st.prefill(x[:40], [40]))
    waited = time.perf_counter() - t0
    arriving = not copies.query()
    torch.cuda.synchronize()
    took = time.perf_counter() - t0
    assert arriving and waited < took / 3, (waited, took)
    assert all(torch.equal(o, want) for o in outs)
    st.close()
