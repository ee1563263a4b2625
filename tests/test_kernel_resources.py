"""What the compiled kernels of libgsr.so hold, from the metadata of the code object built from these sources: no GPU."""
import struct

import msgpack
import pytest

import paper_2603_27156_amd as gsr


def kernels():
    """name -> metadata of every kernel for gfx950 in the library (an offload bundle of ELF code objects per source file)."""
    blob = open(gsr.LIB_PATH, "rb").read()
    magic, at, out = b"__CLANG_OFFLOAD_BUNDLE__", 0, {}
    while (at := blob.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + length].decode()
            p += 24 + length
            if triple.endswith("gfx950"):
                out.update(notes(blob[at + offset:at + offset + size]))
        at += len(magic)
    return out


def notes(elf):
    header, entry, number = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
    found = {}
    for s in range(number):
        kind, _, _, offset, size = struct.unpack_from("<IQQQQ", elf, header + s * entry + 4)
        if kind != 7:                                                # SHT_NOTE
            continue
        name, desc, _ = struct.unpack_from("<III", elf, offset)
        body = elf[offset + 12 + (name + 3) // 4 * 4:][:desc]
        for k in msgpack.unpackb(body).get("amdhsa.kernels", []):
            found[k[".name"]] = k
    return found


def test_no_kernel_spills_registers():
    ks = kernels()
    assert sum("k_block" in n for n in ks) >= 32 and sum("k_grad" in n for n in ks) >= 16
    spilling = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in ks.items()
                if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilling, spilling


# Registers that a launch rule or a measured figure counts on (a wave may have 512 / waves per SIMD of them): two workgroups of eight waves
# beside each other on a compute unit in the products of two and three column blocks, and the sums over neighbours of 32 columns, whose sweep
# slowed by a tenth at 93 registers.
@pytest.mark.parametrize("kernel,most", [
    ("k_wide_productILi2E", 128), ("k_wide_productILi3E", 128), ("k_wide_gradILi2E", 128), ("k_wide_gradILi3E", 128),
    # five workgroups of four waves each (k_dense_planes of 16 bits that deals tiles out holds more and is launched with four)
    ("k_spmm_tile", 96), ("k_aggregate_tile", 96), ("k_gather_wide", 96), ("k_dense_planesIfLb", 96), ("k_dense_planesINS_6bf16_tELb0E", 96),
    ("k_spmm_tileILi32ELb0ELb0E", 80), ("k_spmm_tileILi32ELb1ELb0E", 80),
])
def test_registers_that_residency_counts_on(kernel, most):
    held = {n: k[".vgpr_count"] for n, k in kernels().items() if kernel in n}
    assert held and max(held.values()) <= most, held
