"""The grid of a decode attention launch, on the CPU: every (sequence, kv head, chunk) has a workgroup, and only x, the
dimension that takes them, ever holds more than 65535."""
import ctypes as C

import pytest

from paper_2502_09922_amd import binding


def grid(rows, hkv, nchunk):
    out = (C.c_int * 4)()
    binding.lib.ls_test_attn_decode_grid(rows, hkv, nchunk, C.byref(out))
    return list(out)


@pytest.mark.parametrize("hkv", [1, 4, 8, 40])
@pytest.mark.parametrize("rows", [1, 2, 64, 65535, 65536, 100000, 1 << 20])
def test_sizes(rows, hkv):
    for nchunk in (1, 3, 16):
        x, y, z, heads_first = grid(rows, hkv, nchunk)
        assert (x, y, z) == ((hkv, rows, nchunk) if heads_first else (rows, hkv, nchunk))
        assert y <= 65535 and z <= 65535


@pytest.mark.parametrize("rows", [1, 4, 16, 17, 32, 33, 64, 100])
def test_heads_go_round_the_xcds_but_for_few_sequences_in_chunks(rows):
    assert grid(rows, 8, 1)[3] == 1
    assert grid(rows, 8, 2)[3] == grid(rows, 8, 16)[3] == (0 if rows <= 16 else 1)
    assert grid(rows, 2, 4)[3] == (0 if rows <= 32 else 1)
