"""Scratch memory of the built kernels, from the code objects' own notes: a wavefront that spills registers
goes to memory for them in the middle of its chain of dependent steps."""
import re
import struct

import msgpack

import paper_2411_03357_amd as pgcm

# bytes a lane, of the instances that have any
MOST = {
    r"bulk_kernelILb.ELi(10|14)ELb1E": 80,  # the row hash on the matrix cores
    r"bulk_kernelILb.ELi12ELb1E": 48,
    r"final_kernelILb.E": 12,
    # two workgroups a compute unit have 64 registers a lane; with IVs hashed in rows
    r"burst_kernelILb.ELb1ELNS_9BurstKindE3E": 160,
}


def _code_objects(image):
    """gfx950 ELF images of the bundles in a shared library"""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = image.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", image, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", image, pos)
            target = image[pos + 24:pos + 24 + name]
            pos += 24 + name
            if target.endswith(b"gfx950"):
                yield image[at + offset:at + offset + size]
        at = image.find(magic, pos)


def _kernels(elf):
    """the kernels' entries in the object's metadata note"""
    headers, = struct.unpack_from("<Q", elf, 0x20)
    size, count = struct.unpack_from("<HH", elf, 0x36)
    for i in range(count):
        kind, _, offset, _, _, length = struct.unpack_from("<IIQQQQ", elf, headers + i * size)
        pos, end = offset, offset + length
        while kind == 4 and pos < end:      # PT_NOTE
            names, described, note = struct.unpack_from("<III", elf, pos)
            name = elf[pos + 12:pos + 12 + names].rstrip(b"\0")
            pos += 12 + (names + 3) // 4 * 4
            if name == b"AMDGPU" and note == 32:
                yield from msgpack.unpackb(elf[pos:pos + described])["amdhsa.kernels"]
            pos += (described + 3) // 4 * 4


def test_no_kernel_spills_more_than_known():
    with open(pgcm.library_path(), "rb") as f:
        image = f.read()
    scratch = {k[".name"]: k[".private_segment_fixed_size"] for elf in _code_objects(image) for k in _kernels(elf)}
    for name in ("swap_kernel", "burst_kernel", "span_kernel", "bulk_kernel", "small_kernel", "keystream_kernel"):
        assert any(name in k for k in scratch), (name, len(scratch))
    over = {k: v for k, v in scratch.items()
            if v > max([0] + [most for pattern, most in MOST.items() if re.search(pattern, k)])}
    assert not over, over
