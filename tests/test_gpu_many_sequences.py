"""Generation steps of more sequences than a launch takes in y or z (65535), short contexts: against the same step in two
halves, of whose row counts every kernel has tests of its own."""
import pytest

import synth
from helpers import make_gpu, to_dev
from paper_2502_09922_amd import binding  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [synth.StageShape("bf16", 1, 64, 1, 1, 64, 64, 0), synth.StageShape("f32", 1, 64, 2, 1, 64, 64, 0),
                                   synth.StageShape("bf16", 1, 128, 2, 1, 128, 128, 0)], ids=["mha", "f32", "gqa"])
def test_70000_sequences(shape):
    import torch

    n, half, room, ctx = 70000, 35000, 8, 5
    gen = torch.Generator(device="cuda").manual_seed(1)
    gpu = make_gpu(shape, 1, 0, 1, n, room, n)
    x = torch.randn(n, shape.hidden, generator=gen, device="cuda").to(gpu.tdtype)
    lens = torch.randint(1, ctx + 1, (n,), generator=gen, device="cuda", dtype=torch.int32)
    k = [torch.randn(n * room * shape.n_kv_heads * shape.head_dim, generator=gen, device="cuda").to(gpu.tdtype) for _ in range(2)]
    per = k[0].numel() // n
    gpu.seq_lens.copy_(lens)
    gpu.k.view(gpu.tdtype).copy_(k[0])
    gpu.v.view(gpu.tdtype).copy_(k[1])
    got = gpu.decode(x, n, ctx)
    assert torch.equal(gpu.seq_lens, lens + 1)
    ref = make_gpu(shape, 1, 0, 1, half, room, half)
    for a in (0, half):
        ref.seq_lens.copy_(lens[a : a + half])
        ref.k.view(gpu.tdtype).copy_(k[0][a * per : (a + half) * per])
        ref.v.view(gpu.tdtype).copy_(k[1][a * per : (a + half) * per])
        want = ref.decode(x[a : a + half], half, ctx)
        err = ((got[a : a + half].double() - want.double()).norm() / want.double().norm()).item()
        # other tiles may add up in another order: 2^-9 of a bf16 value, some 2^-24 of an fp32 one
        assert err <= (2.0**-8 if shape.dtype == "bf16" else 1e-5), (a, err)
    ref.close()
    gpu.close()
