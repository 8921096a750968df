"""Scratch memory of the built kernels, from the metadata of the code objects in libbns.so: only kernels that the build allows use any."""
import os
import struct
import sys

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)
import __graft_entry__ as entry  # noqa: E402

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(library):
    """The device code objects of every bundle in the library."""
    at = library.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", library, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", library, pos)
            triple = library[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in triple:
                yield library[at + offset:at + offset + size]
        at = library.find(MAGIC, at + 1)


def _kernels(elf):
    """{mangled name: bytes of scratch memory per lane} of an ELF code object (note type 32, "AMDGPU": a msgpack map)."""
    assert elf[:4] == b"\x7fELF"
    (phoff,), (phentsize, phnum) = struct.unpack_from("<Q", elf, 32), struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
        if kind != 4:                                       # PT_NOTE
            continue
        pos, end = offset, offset + size
        while pos < end:
            name_size, desc_size, note = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (name_size + 3) // 4 * 4
            if note == 32 and elf[pos + 12:pos + 18] == b"AMDGPU":
                meta = msgpack.unpackb(elf[desc:desc + desc_size])
                return {k[".name"]: k[".private_segment_fixed_size"] for k in meta["amdhsa.kernels"]}
            pos = desc + (desc_size + 3) // 4 * 4
    return {}


def test_only_the_kernels_that_the_build_allows_use_scratch_memory():
    if not os.path.exists(entry.LIB):
        pytest.skip("libbns.so is not built")
    kernels = {}
    for elf in _code_objects(open(entry.LIB, "rb").read()):
        kernels.update(_kernels(elf))
    assert sum("nhwc_fused_backward_kernel" in name for name in kernels) > 20 and sum("resident_" in name for name in kernels) == 40
    assert entry.unexpected_scratch(kernels) == {}


def test_a_kernel_that_is_not_listed_or_needs_more_is_reported():
    listed = "_ZN3bns12_GLOBAL__N_126fused_backward_pipe_kernelINS_6bf16_tELi8ELi5ELi512EEEvNS0_9FusedArgsE"
    other = listed.replace("Li5E", "Li4E")
    remark = "x.hip:1:1: remark: {} [-Rpass-analysis=kernel-resource-usage]"
    report = "\n".join([remark.format("Function Name: " + listed), "source", "^", remark.format("    ScratchSize [bytes/lane]: 16"),
                        remark.format("Function Name: " + other), "source", "^", remark.format("    ScratchSize [bytes/lane]: 4"), "a warning"])
    lines, spilled = entry._split_resource_remarks(report)
    assert lines == ["a warning"] and spilled == {listed: 16, other: 4}
    assert entry.unexpected_scratch(spilled) == {other: 4}
    assert entry.unexpected_scratch({listed: 60}) == {listed: 60}
