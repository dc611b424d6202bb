"""What the compiler made of the kernels, read from the code objects inside the built library (kernel metadata, AMDGPU notes): the
GEMM tiles, the row kernel and the decode attention of grouped queries keep everything in registers."""
import re
import struct

import msgpack

from paper_2502_09922_amd import binding

# 128 and more fp32 values of eight query heads, weights 16 k-steps ahead, 512-register tiles: spilled since they were written
KNOWN = ("k_attn_decodeIfLi128ELi8E", "k_attn_decodeIfLi64ELi8E", "k_attn_decodeIDF16bLi128ELi8E", "k_attn_decodeIDF16bLi64ELi8E",
         "k_gemm_mfma", "k_gemm_skinnyILi1ELi2ELi16E", "k_gemm_skinnyILi4ELi2ELi8E")


def kernels():
    data, out, at = open(binding.LIB_PATH, "rb").read(), {}, 0
    while (at := data.find(b"\x7fELF\x02\x01\x01\x40", at)) >= 0:  # 64 bits, little-endian, AMDGPU HSA
        shoff, = struct.unpack_from("<Q", data, at + 40)
        size, count = struct.unpack_from("<HH", data, at + 58)
        for i in range(count):
            kind, = struct.unpack_from("<I", data, at + shoff + i * size + 4)
            offset, = struct.unpack_from("<Q", data, at + shoff + i * size + 24)
            if kind == 7:  # notes
                name, desc, note = struct.unpack_from("<III", data, at + offset)
                if note == 32:
                    start = at + offset + 12 + (name + 3) // 4 * 4
                    for k in msgpack.unpackb(data[start : start + desc])["amdhsa.kernels"]:
                        out[k[".name"]] = k
        at += 4
    return out


def test_no_kernel_spills_that_did_not():
    found = kernels()
    assert len(found) > 200 and sum("k_gemm_tiled" in n for n in found) > 80
    spilled = {n: (k[".vgpr_count"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in found.items()
               if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not [n for n in spilled if not any(re.search(k, n) for k in KNOWN)], spilled
