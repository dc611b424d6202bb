"""Grouped-query decode attention gives its workgroups the sequences by length: every sequence has to be taken, and once,
whatever the lengths: ties, all alike, in order and against it, sequences without room, more than the workgroups that
fit the chip at once, the most that are ordered and one more."""
import numpy as np
import pytest

import synth
from helpers import check_close, make_gpu, make_oracle, to_dev, to_host

pytestmark = pytest.mark.gpu

SHAPE = synth.StageShape("bf16", 1, 256, 8, 4, 128, 256, 0)


@pytest.mark.parametrize("batch", [2, 3, 63, 64, 65, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("order", ["random", "alike", "up", "down"])
def test_every_sequence_is_taken_once(batch, order):
    rng = np.random.default_rng(batch)
    room = 48
    lengths = [int(n) for n in rng.integers(1, room + 1, size=batch)]  # a sequence of `room` tokens has no room for another
    if order == "alike":
        lengths = [17] * batch
    elif order != "random":
        lengths = sorted(lengths, reverse=order == "down")
    gpu, ora = make_gpu(SHAPE, 1, 0, 1, batch, room, sum(lengths)), make_oracle(SHAPE, 1, 0, 1, batch, room)
    x, xs = synth.hidden_states(SHAPE, 2, sum(lengths)), synth.hidden_states(SHAPE, 3, batch)
    gpu.prefill(to_dev(SHAPE, x), lengths)
    ora.prefill(x, lengths)
    live = [i for i, n in enumerate(lengths) if n < room]
    got = to_host(gpu.decode(to_dev(SHAPE, xs), batch, min(max(lengths), room - 1)))
    for i, n in enumerate(lengths):
        if n == room:
            ora.seq_lens[i] = 1  # its row is not compared
    want = ora.decode(xs)
    check_close(got[live], want[live], "bf16", "%d sequences, %s" % (batch, order))
    assert gpu.seq_lens.cpu().tolist() == [min(n + 1, room) for n in lengths]
    gpu.close()
