"""What the built kernels ask for, read from the code objects in the library (no GPU needed)."""
import os
import re
import struct

import pytest

from paper_2110_03423_amd import binding

LDS_PER_CU, WAVES_PER_SIMD = 160 * 1024, 8


def _kernels():
    """Metadata of every kernel: the note of each gfx950 code object in the library's offload bundles."""
    msgpack = pytest.importorskip("msgpack")
    if not os.path.exists(binding.library_path()):
        from paper_2110_03423_amd import build
        build.build_library()
    blob = open(binding.library_path(), "rb").read()
    out, magic, at = {}, b"__CLANG_OFFLOAD_BUNDLE__", -1
    while (at := blob.find(magic, at + 1)) >= 0:
        entries, pos = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(entries):
            offset, size, name = struct.unpack_from("<QQQ", blob, pos)
            target = blob[pos + 24:pos + 24 + name]
            pos += 24 + name
            if b"gfx950" not in target or size == 0:
                continue
            elf = blob[at + offset:at + offset + size]
            note = elf.find(b"AMDGPU\0\0")
            length = struct.unpack_from("<I", elf, note - 8)[0]
            meta = msgpack.unpackb(elf[note + 8:note + 8 + length])
            out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
    return out


def test_small_svd_kernels_leave_room_for_the_problems_of_a_batch():
    """Without the corrections of the whole matrix a CU holds as many problems as its LDS (or its wavefront slots) does: the registers
    are not what limits them."""
    seen = set()
    for name, k in _kernels().items():
        m = re.search(r"jacobi_lds_kernelI([fd])[fd]Li(\d+)ELi16ELb(\d)E(?:Lb(\d)E)?", name)
        if not m or m[3] == "1" or m[4] == "1":           # (J in global memory: no batch of these has two problems to a CU; with corrections)
            continue
        size, rpl = {"f": 4, "d": 8}[m[1]], int(m[2])
        seen.add((size, rpl))
        assert k[".vgpr_spill_count"] == 0 and k[".sgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, name
        waves = 4 * min(WAVES_PER_SIMD, 512 // (-(-k[".vgpr_count"] // 8) * 8))
        step = 16 * (8 // size)
        for l in range(max(2, 16 * (rpl - 1) - 15), 16 * rpl + 1):
            rows = -(-l // step) * step
            if rows != 16 * rpl:
                continue
            lds = 2 * l * (rows + 2) * size + l * (size + 4) + k[".group_segment_fixed_size"]
            mine = -(-(l + 1) // 2 * 16 // 64)
            assert waves // mine >= min(LDS_PER_CU // lds, 4 * WAVES_PER_SIMD // mine), (name, l)
    assert {(4, 2), (4, 4), (4, 6), (4, 8), (8, 1), (8, 2), (8, 3), (8, 4), (8, 5), (8, 6)} <= seen
