"""The sequence bounds of a prompt pass: written in stream order on the current stream (more of them than one kernel
carries), copied where the pass runs on another stream or reads rows in pinned host memory; passes one behind the other with nothing
waited for between them."""
import ctypes as C

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
    gpu.prefill(to_dev(shape, synth.hidden_states(shape, 9, 3)), [3])  # the first behind a load copies its bounds
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
