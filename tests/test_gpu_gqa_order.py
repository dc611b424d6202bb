"""Grouped-query decode attention gives its workgroups the sequences by length where contexts may be long: every sequence has
to be taken, and once, whatever the lengths: ties, all alike, in order and against it, sequences without room, as
many as fit the chip at once (64 of 8 kv heads) and more, the most that are ordered and one more.  Fewer sequences are
cut into chunks, and short contexts are taken in the order of the rows."""
import numpy as np
import pytest

import synth
from helpers import check_close, make_gpu, make_oracle, to_dev, to_host

pytestmark = pytest.mark.gpu

SHAPE = synth.StageShape("bf16", 1, 256, 16, 8, 128, 256, 0)
ROOM = 560


CASES = [(b, o, 559) for b in (2, 3, 63, 64, 65, 128, 129, 193, 255, 256, 257) for o in ("random", "alike", "up", "down")]
CASES += [(b, "random", c) for b in (64, 256) for c in (40, 511, 512)]


@pytest.mark.parametrize("batch,order,max_ctx", CASES)
def test_every_sequence_is_taken_once(batch, order, max_ctx):
    rng = np.random.default_rng(batch)
    lengths = [int(n) for n in rng.integers(1, 17, size=batch)]
    if order == "alike":
        lengths = [11] * batch
    elif order != "random":
        lengths = sorted(lengths, reverse=order == "down")
    gpu, ora = make_gpu(SHAPE, 1, 0, 1, batch, ROOM, sum(lengths)), make_oracle(SHAPE, 1, 0, 1, batch, ROOM)
    x, xs = synth.hidden_states(SHAPE, 2, sum(lengths)), synth.hidden_states(SHAPE, 3, batch)
    gpu.prefill(to_dev(SHAPE, x), lengths)
    ora.prefill(x, lengths)
    full = [i for i in range(batch) if i % 7 == 3 and order != "alike"]  # sequences without room for another row
    for i in full:
        gpu.seq_lens[i] = ROOM
    live = [i for i in range(batch) if i not in full]
    got = to_host(gpu.decode(to_dev(SHAPE, xs), batch, max_ctx))
    want = ora.decode(xs)
    check_close(got[live], want[live], "bf16", "%d sequences, %s" % (batch, order))
    assert gpu.seq_lens.cpu().tolist() == [ROOM if i in full else n + 1 for i, n in enumerate(lengths)]
    gpu.close()


def test_ordering_costs_less_than_it_can_gain():
    """Finding the order is work of every workgroup: with it 256 sequences may not take longer than 257, which are taken
    in the order of the rows (ranks through LDS: 132 us against 105)."""
    import torch

    gpu = make_gpu(synth.StageShape("bf16", 1, 2048, 16, 8, 128, 256, 0), 1, 0, 1, 257, ROOM, 257)
    lens = torch.full((257,), 250, dtype=torch.int32, device="cuda")
    x = torch.randn(257, 2048, device="cuda").to(torch.bfloat16)
    best = {}
    for _ in range(5):
        for rows in (256, 257):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            for i in range(25):
                if i == 5:
                    a.record()
                gpu.seq_lens.copy_(lens)
                gpu.decode(x[:rows], rows, 559)
            b.record()
            torch.cuda.synchronize()
            best[rows] = min(best.get(rows, 1e9), a.elapsed_time(b) / 20)
    gpu.close()
    print("256 sequences %.1f us, 257 %.1f us" % (1e3 * best[256], 1e3 * best[257]))
    assert best[256] <= 1.12 * best[257]
