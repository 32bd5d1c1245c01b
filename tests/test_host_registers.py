"""Registers of the built kernels, from the code objects' own metadata: a launch that counts on two blocks of four waves per CU
gets them only while a wave takes at most 256 of a SIMD's 512 registers."""
import struct

import msgpack

from paper_2511_10333_amd import binding


def _kernels():
    """{mangled name: metadata} of every gfx950 kernel in libedgc.so (clang offload bundles of ELF objects, each with an AMDGPU
    metadata note in MessagePack)."""
    so, out, at = open(binding.lib_path(), "rb").read(), {}, 0
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    while (at := so.find(magic, at)) >= 0:
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", so, at + len(magic))[0]):
            offset, size, length = struct.unpack_from("<QQQ", so, pos)
            target = so[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" not in target:
                continue
            elf = so[at + offset:at + offset + size]
            note = elf.find(struct.pack("<I", 32) + b"AMDGPU\0\0")      # type 32: metadata
            if note >= 0:
                desc = struct.unpack_from("<I", elf, note - 4)[0]
                meta = msgpack.unpackb(elf[note + 12:note + 12 + desc])
                out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
        at += len(magic)
    return out


def test_two_blocks_of_the_p_pass_share_a_cu():
    found = {n: k for n, k in _kernels().items() if "8k_pass_pI" in n}
    assert len(found) >= 6                                              # one or two planes, one, two or four tiles of rank
    for name, k in found.items():
        assert k[".vgpr_count"] <= 256 and k[".vgpr_spill_count"] == 0, (name, k[".vgpr_count"], k[".vgpr_spill_count"])
