"""Keys to a tile of bf16 prompt attention, on the CPU: 32 only with head_dim 128, workgroups beyond what the chip holds at once
and a head of a sequence for each CU; rows are counted, not the grid of the longest prompt."""
from paper_2502_09922_amd import binding


def keys(hq, hd, lengths):
    return binding.lib.ls_test_attn_prefill_keys(hq, hd, len(lengths), sum(lengths))


def test_rule():
    assert keys(40, 128, [1024] * 32) == keys(64, 128, [2048, 1800, 1500, 1200, 600, 148]) == keys(32, 128, [512] * 8) == 32
    # few sequences of many tiles, and too few rows for the chip
    assert keys(40, 128, [2048]) == keys(64, 128, [2048]) == keys(40, 128, [1024] * 4) == keys(32, 128, [311]) == 64
    assert keys(32, 128, [64] * 8) == keys(8, 128, [128] * 32) == 64
    # one long prompt beside short ones: a grid of 5120 workgroups, most of which leave at once
    assert keys(40, 128, [2048] + [300] * 5) == 64
    assert keys(32, 64, [1024] * 32) == 64
    # at the limits
    assert keys(32, 128, [512] * 7 + [511]) == 32 and keys(32, 128, [586] * 7) == 64
    assert keys(128, 128, [192, 192]) == 64 and keys(128, 128, [193, 192]) == 32


def test_largest_shapes_do_not_overflow():
    assert binding.lib.ls_test_attn_prefill_keys(1 << 14, 128, 1 << 16, 1 << 30) == 32
