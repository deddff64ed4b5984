"""What the built library's code objects say of the kernels' registers (host only): the kernels whose
key buffers live on from one chunk of rows to the next must hold them in registers."""
import re
import struct

import msgpack

import paper_2408_00167_amd as F


def _notes(elf):
    """Descriptors of the AMDGPU metadata notes (type 32) of one code object."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, = struct.unpack_from("<I", elf, phoff + i * phentsize)
        offset, = struct.unpack_from("<Q", elf, phoff + i * phentsize + 8)
        size, = struct.unpack_from("<Q", elf, phoff + i * phentsize + 32)
        at = offset
        while kind == 4 and at < offset + size:  # PT_NOTE
            namesz, descsz, note = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if note == 32 and elf[at + 12:at + 18] == b"AMDGPU":
                yield elf[desc:desc + descsz]
            at = desc + (descsz + 3) // 4 * 4


def kernels():
    """{mangled name: metadata} of every kernel in libfinch.so."""
    F.load_library()
    with open(F.LIB_PATH, "rb") as f:
        data = f.read()
    out = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        base = m.start()
        count, = struct.unpack_from("<Q", data, base + 24)
        at = base + 32
        for _ in range(count):
            offset, size, idlen = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" in triple:
                for note in _notes(data[base + offset:base + offset + size]):
                    for k in msgpack.unpackb(note)["amdhsa.kernels"]:
                        out[k[".name"]] = k
    return out


def test_document_row_kernels_keep_their_key_buffers_in_registers():
    """At most four 4-byte values a lane are spilled (values set once per launch and read once per step);
    a key buffer of 128 channels is 32."""
    seen = 0
    for name, meta in kernels().items():
        m = re.search(r"owner_(step|loop)_bf16ILi(\d+)ELi(\d+)ELb([01])ELb1E", name)
        if m:
            seen += 1
            assert meta[".vgpr_spill_count"] <= 4, f"{m.groups()}: {meta['.vgpr_spill_count']} spilled"
    assert seen == 32  # step and loop, 2 head sizes, 4 numbers of row blocks, with re-positioning and without


def test_row_statistics_of_many_rows_are_not_spilled():
    """More than 256 rows of 128 channels leave room for one workgroup a compute unit: twice the registers."""
    seen = 0
    for name, meta in kernels().items():
        m = re.search(r"rowstats_bf16ILi(\d+)ELi(12|16)E", name)
        if m:
            seen += 1
            assert meta[".vgpr_spill_count"] == 0, f"{m.groups()}: {meta['.vgpr_spill_count']} spilled"
    assert seen == 4


def test_one_pass_loops_keep_their_key_buffers_in_registers():
    """At most four 4-byte values a lane are spilled, as above."""
    seen = 0
    for name, meta in kernels().items():
        m = re.search(r"owner_loop_bf16ILi(\d+)ELi(\d+)ELb([01])ELb0ELb1E", name)
        if m:
            seen += 1
            assert meta[".vgpr_spill_count"] <= 4, f"{m.groups()}: {meta['.vgpr_spill_count']} spilled"
    assert seen == 16  # 2 head sizes, 4 numbers of row blocks, with re-positioning and without
