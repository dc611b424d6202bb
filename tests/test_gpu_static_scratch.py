"""The static array behind ls_stage_decode_static is shared by all stages of a device, so only the steps that
ls_stage.h names (bf16, 17..64 rows) may write it: those of other sizes and of fp32 leave it as it is, and give what
ls_stage_decode gives."""
import ctypes as C

import pytest
import torch

import synth
from helpers import make_gpu, to_dev

pytestmark = pytest.mark.gpu

S = synth.StageShape
MARK = 0x5A


def static_array():
    from paper_2502_09922_amd import binding

    fn = binding.lib.ls_test_static_scratch
    fn.restype = C.c_void_p
    n = 16 << 20  # LS_STATIC_SCRATCH_BYTES

    class Array:
        __cuda_array_interface__ = dict(shape=(n,), typestr="|u1", data=(fn(), False), version=2)

    return torch.as_tensor(Array(), device="cuda")


@pytest.mark.parametrize("shape,batch,shared", [
    (S("f32", 1, 1024, 4, 4, 64, 1408, 0), 3, False),  # few rows, K cut
    (S("f32", 1, 1024, 4, 4, 64, 1408, 0), 33, False),
    (S("bf16", 1, 5120, 4, 4, 128, 1408, 0), 12, False),  # wide layers: the tiled GEMM from 9 rows on
    (S("bf16", 1, 1024, 4, 4, 64, 1408, 0), 65, False),
    (S("bf16", 1, 1024, 4, 4, 64, 1408, 0), 100, False),
    (S("bf16", 1, 1024, 4, 4, 64, 1408, 0), 64, True),
])
def test_which_steps_write_the_static_array(shape, batch, shared):
    gpu = make_gpu(shape, 3, 0, 1, batch, 8, batch)
    x = to_dev(shape, synth.hidden_states(shape, 4, batch))
    gpu.prefill(x, [1] * batch)
    want = gpu.decode(x, batch, 1).clone()
    array = static_array()
    array.fill_(MARK)
    gpu.seq_lens.fill_(1)
    got = gpu.decode(x, batch, 1, static=True)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert bool((array != MARK).any()) == shared
    gpu.close()
