"""Register use of the built kernels, read from the metadata of the library's
gfx950 code objects (no GPU)."""
import os
import struct

import msgpack

import paper_2607_08643_amd as bsq

AMDGPU_ELF = b"\x7fELF\x02\x01\x01\x40"  # 64-bit little-endian, OS ABI 64 (AMDGPU HSA)
NT_AMDGPU_METADATA, SHT_NOTE = 32, 7


def kernels():
    """The metadata of every kernel in the library, by symbol name."""
    path = os.path.join(os.path.dirname(bsq.__file__), "libbsq.so")
    with open(path, "rb") as f:
        data = f.read()
    out, at = {}, data.find(AMDGPU_ELF)
    while at >= 0:
        elf = data[at:]
        shoff, = struct.unpack_from("<Q", elf, 0x28)
        size, count = struct.unpack_from("<HH", elf, 0x3A)
        for i in range(count):
            _, kind, _, _, off, length = struct.unpack_from("<IIQQQQ", elf, shoff + i * size)
            end = off + length
            while kind == SHT_NOTE and off < end:
                name, desc, note = struct.unpack_from("<III", elf, off)
                body = off + 12 + (name + 3) // 4 * 4
                if note == NT_AMDGPU_METADATA:
                    for k in msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]:
                        out[k[".name"]] = k
                off = body + (desc + 3) // 4 * 4
        at = data.find(AMDGPU_ELF, at + 4)
    return out


def test_topk_keys_stay_in_registers():
    """The selection's register runs (8, 16 and 32 keys a thread, 1024 threads)
    fit the 128 registers of a lane: no scratch memory."""
    topk = {n: k for n, k in kernels().items() if "topk_kernel" in n}
    assert len(topk) == 4
    for name, k in topk.items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name
