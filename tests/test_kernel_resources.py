"""No kernel of the library uses scratch memory: the header promises that nothing is allocated on a call's behalf, and the
runtime allocates scratch for a queue when a kernel that spills registers first runs on it.  Read from the metadata of
the built library's own code objects (host only)."""
import struct

import msgpack


def code_objects(blob):
    """The gfx950 code objects of every offload bundle in a shared library."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + length]:
                yield blob[at + offset:at + offset + size]
            p += 24 + length
        at += len(magic)


def kernels(elf):
    """The kernels of a code object: the msgpack note NT_AMDGPU_METADATA (32)."""
    (shoff,) = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        offset, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        end = offset + size
        while kind == 7 and offset < end:
            namesz, descsz, note = struct.unpack_from("<III", elf, offset)
            desc = offset + 12 + (namesz + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[desc:desc + descsz]).get("amdhsa.kernels", [])
            offset = desc + (descsz + 3) // 4 * 4


def test_no_kernel_uses_scratch():
    from paper_2005_09904_amd.build import LIB_PATH

    with open(LIB_PATH, "rb") as f:
        found = {k[".name"]: k for elf in code_objects(f.read()) for k in kernels(elf)}
    assert len(found) > 100                              # (the notes were found)
    spilled = {n: k[".private_segment_fixed_size"] for n, k in found.items() if k[".private_segment_fixed_size"]
               or k.get(".uses_dynamic_stack")}
    assert not spilled


def test_gather8_without_a_loop_over_splits_is_compiled_without_one():
    """Where the grid holds the splits, the compiler has to see that a wave has one of them: kept as a loop, the addresses of all
    its reads stay in registers, as many as where a wave does have several."""
    from paper_2005_09904_amd.build import LIB_PATH

    with open(LIB_PATH, "rb") as f:
        vgprs = {k[".name"]: k[".vgpr_count"] for elf in code_objects(f.read()) for k in kernels(elf) if "gather8_kernel" in k[".name"]}
    single = [n for n in vgprs if "ELb0EEEv" in n]
    assert len(single) == 24 and len(vgprs) == 48        # planes, both orders, slices on neighbouring lanes
    for n in single:
        assert vgprs[n] < 0.9 * vgprs[n.replace("ELb0EEEv", "ELb1EEEv")], (n, vgprs[n])
