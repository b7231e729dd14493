"""The kernels of the built library, from the metadata of its own code objects.  The register tiles of the tiled
kernels stay in registers: their scratch memory holds spilled registers and nothing else (a tile array indexed at
run time, or a function call, would add hundreds of bytes).  And no kernel is compiled that no call launches."""
import os
import re
import struct

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(__file__), "..", "paper_2403_07412_amd", "libvecchia.so")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """AMDGPU metadata notes (type 32) of a code object."""
    table, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        _, kind, _, _, at, size = struct.unpack_from("<IIQQQQ", elf, table + k * entry)
        end = at + size
        while kind == 7 and at < end:  # SHT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if note == 32:
                yield msgpack.unpackb(elf[at:at + desc])
            at += (desc + 3) // 4 * 4


def _kernels():
    with open(LIB, "rb") as f:
        data = f.read()
    at = data.find(BUNDLE)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + len(BUNDLE))
        p = at + len(BUNDLE) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                for note in _notes(data[at + offset:at + offset + size]):
                    yield from note["amdhsa.kernels"]
            p += 24 + length
        at = data.find(BUNDLE, at + 1)


def test_tiles_are_not_in_scratch_memory():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    kernels = [k for k in _kernels() if "cond_kernel" in k[".name"] or "cond_group_kernel" in k[".name"]]
    assert kernels
    bad = [(k[".name"], k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in kernels
           if k[".private_segment_fixed_size"] > 4 * k[".vgpr_spill_count"] + 16 or k.get(".uses_dynamic_stack")]
    assert not bad


def test_no_tiled_kernel_where_the_rows_kernel_runs():
    """One wavefront, up to four tile rows (codes 0 .. 2) or two (3 .. 7): only the rows kernel is compiled."""
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    shapes = [tuple(map(int, m.groups())) for m in
              (re.search(r"TileImplILi(\d+)ELi(\d+)ELi(\d+)E", k[".name"]) for k in _kernels()) if m]
    assert shapes
    assert not [s for s in shapes if s[1] == 1 and s[0] <= (4 if s[2] < 3 else 2)]


def test_eight_tile_rows_run_four_workgroups():
    """Eight tile rows by four wavefronts: up to 128 registers hold four workgroups per compute unit, 129 three."""
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    regs = {k[".name"]: k[".vgpr_count"] for k in _kernels() if "TileImplILi8ELi4E" in k[".name"]}
    assert len(regs) == 16 and max(regs.values()) <= 128, regs
