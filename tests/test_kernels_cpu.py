"""What the compiler made of the kernels: the metadata of the built code object."""
import os
import re
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def kernels(qtn):
    """Kernel name -> metadata, from the notes of every gfx950 code object."""
    with open(os.path.join(ROOT, "paper_2204_06045_amd", "libqtn.so"), "rb") as f:
        lib = f.read()
    out = {}
    for at in [m.start() for m in re.finditer(b"\x7fELF", lib)][1:]:
        elf = lib[at:]
        phoff, = struct.unpack_from("<Q", elf, 32)
        phsize, phnum = struct.unpack_from("<HH", elf, 54)
        for k in range(phnum):
            kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + k * phsize)
            end = off + size
            while kind == 4 and off + 12 <= end:  # PT_NOTE
                name, desc, _ = struct.unpack_from("<III", elf, off)
                body = off + 12 + (name + 3) // 4 * 4
                if elf[off + 12:off + 12 + name] == b"AMDGPU\0":
                    meta = msgpack.unpackb(elf[body:body + desc])
                    out.update({x[".name"]: x for x in meta["amdhsa.kernels"]})
                off = body + (desc + 3) // 4 * 4
    assert out
    return out


def test_cell_kernels_hold_their_cells_in_registers(kernels):
    """No cell kernel keeps its accumulators in scratch memory (2^CB cells of 8
    or 16 bytes, a good part of which an indexed array would put there); the
    ones in the plan's order use none at all."""
    seen = 0
    for name, meta in kernels.items():
        m = re.search(r"k_wide_cellsI15HIP_vector_typeI([fd])Lj2EELb[01]ELi(\d)ELi(\d)ELb([01])E", name)
        if not m:
            continue
        seen += 1
        cells = (8 if m[1] == "f" else 16) << int(m[2])
        scratch = meta[".private_segment_fixed_size"]
        assert scratch <= (0 if m[4] == "1" else cells // 4), (name, scratch)
    assert seen >= 36
