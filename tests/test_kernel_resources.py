"""What the compiled kernels of libgsr.so hold, from the metadata of the code object built from these sources: no GPU."""
import struct

import msgpack

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
