"""What the one-launch generation steps of small fp32 models keep between them is no one else's: stages that take turns on one
workspace, a workspace written between steps, more stages than the library has room for, steps on several streams at once."""
import pytest

import synth
from helpers import make_gpu, packed_blocks
from paper_2502_09922_amd import binding as b

pytestmark = pytest.mark.gpu

SHAPE = synth.StageShape("f32", 2, 128, 2, 2, 64, 256, 96)


def small_steps():
    b.lib.ls_test_small_steps.restype = b.C.c_long
    return b.lib.ls_test_small_steps()


def make_stages(spans, shared):
    """Stages of two sequences, each with a workspace of its own or all with the largest one."""
    stages = [make_gpu(SHAPE, 5, lo, hi, 2, 64, 40, load=False) for lo, hi in spans]
    big = max((st.workspace for st in stages), key=lambda t: t.numel())
    for st in stages:
        if shared:
            b.lib.ls_stage_destroy(st.handle)
            st.workspace = big
            b.check(b.lib.ls_stage_create(b.C.byref(st.cfg), st.lo, st.hi, st.slab.data_ptr(), st.slab.numel(), big.data_ptr(), big.numel(), b.C.byref(st.handle)))
        for layer, buf in packed_blocks(st, 5).items():
            st.load_block(layer, st.stage_host_block(layer, buf))
    return stages


def run(stages, steps, between=lambda: None):
    """Outputs of a prompt and `steps` steps through the stages in turn."""
    import torch

    torch.cuda.synchronize()
    outs = []
    rows = torch.randint(0, SHAPE.vocab, (33,), dtype=torch.int32, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    for st in stages:
        rows = st.prefill(rows, [30, 3])
    for t in range(steps):
        for st in stages:
            rows = st.decode(rows, 2, 30 + t)
            outs.append(rows.clone())
            between()
    return outs


def same(got, want):
    import torch

    assert len(got) == len(want) and all(torch.equal(x, y) for x, y in zip(got, want))


def close(stages):
    for st in stages:
        st.close()


def test_stages_take_turns_on_one_workspace():
    own, one = make_stages([(0, 1), (1, 2)], False), make_stages([(0, 1), (1, 2)], True)
    want, before = run(own, 12), small_steps()
    same(run(one, 12), want)
    assert small_steps() == before + 24
    close(own + one)


def test_a_workspace_written_between_steps():
    import torch

    st = make_gpu(SHAPE, 5, 0, 2, 2, 64, 40)
    want, before = run([st], 8), small_steps()
    table = 64 * 32 * 2 * 4  # positions, pairs of a head, cos and sin, fp32
    value = iter(range(100))
    same(run([st], 8, lambda: st.workspace[table:].view(torch.int32).fill_(next(value))), want)
    assert small_steps() == before + 8
    close([st])


def test_stages_beyond_the_librarys_room():
    first = make_stages([(0, 2)] * 70, False)
    want, before = run([first[0]], 3), small_steps()
    for st in first[1:]:
        same(run([st], 3), want)
    taken = small_steps() - before
    assert taken % 3 == 0 and taken <= 63 * 3  # stages of other tests that are still to be collected may hold some
    close(first[:2])
    more = make_stages([(0, 2)], False)
    before = small_steps()
    same(run(more, 3), want)
    assert small_steps() == before + 3
    close(first + more)


def test_steps_on_several_streams_at_once():
    import torch

    stages = make_stages([(0, 2)] * 6, False)
    want = run([stages[0]], 20)
    prompt = torch.randint(0, SHAPE.vocab, (33,), dtype=torch.int32, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    tokens = [st.prefill(prompt, [30, 3]) for st in stages]
    torch.cuda.synchronize()
    streams, before = [torch.cuda.Stream() for _ in stages], small_steps()
    outs = [[torch.empty(2, dtype=torch.int32, device="cuda") for _ in want] for _ in stages]
    for t in range(len(want)):
        for st, stream, out, first in zip(stages, streams, outs, tokens):
            st.decode(out[t - 1] if t else first, 2, 30 + t, stream=stream, out=out[t])
    torch.cuda.synchronize()
    for out in outs:
        same(out, want)
    assert small_steps() == before + 20 * 6
    close(stages)


def test_streams_restricted_to_few_cus_take_separate_launches():
    import ctypes

    import torch

    hip = ctypes.CDLL([l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l][0])  # the one torch uses
    own = make_stages([(0, 2)], False)
    want = run(own, 6)
    few, enough, odd = (1 << 16) - 1, (1 << 24) - 1, 0xFFFF0FFF
    for words, one_launch in (([few] * 8, False), ([enough] * 8, True), ([odd] * 8, True), ([0xFFFFFFFF] * 7 + [few], False), ([0xFFFFFFFF] * 8, True)):
        handle = ctypes.c_void_p()
        mask = (ctypes.c_uint32 * 8)(*words)
        assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, mask) == 0
        stream, before = torch.cuda.ExternalStream(handle.value), small_steps()
        with torch.cuda.stream(stream):
            own[0].reset_blocks()
            for layer in own[0].block_ids():
                own[0].adopt_block(layer, stream)
            stream.synchronize()
            rows = torch.randint(0, SHAPE.vocab, (33,), dtype=torch.int32, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
            rows, got = own[0].prefill(rows, [30, 3], stream=stream), []
            for t in range(6):
                rows = own[0].decode(rows, 2, 30 + t, stream=stream)
                got.append(rows.clone())
        stream.synchronize()
        same(got, want)
        assert small_steps() - before == (6 if one_launch else 0)
        assert hip.hipStreamDestroy(handle) == 0
    close(own)
