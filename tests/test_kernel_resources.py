"""What the compiler gave the kernels of the built library, from the code objects' own metadata."""
import os
import struct

import msgpack

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1108_4214_amd", "libdynbond.so")
BOX_BYTES = 112   # sizeof(Box)


def _kernels():
    """name -> metadata of every GPU kernel: the code objects lie in the library as offload bundles (a table of offset,
    size and target), each an ELF file whose AMDGPU note (type 32) is a msgpack map"""
    data = open(LIB, "rb").read()
    out, at = {}, data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, n = struct.unpack_from("<3Q", data, p)
            target = data[p + 24:p + 24 + n]
            p += 24 + n
            if target.startswith(b"hip") and size:
                out.update(_notes(data[at + offset:at + offset + size]))
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    return out


def _notes(elf):
    assert elf[:4] == b"\x7fELF"
    sections, entry, count = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<2H", elf, 58)
    for k in range(count):
        kind, offset, size = (struct.unpack_from(f, elf, sections + k * entry + o)[0]
                              for f, o in (("<I", 4), ("<Q", 24), ("<Q", 32)))
        while kind == 7 and size >= 12:
            name, desc, note = struct.unpack_from("<3I", elf, offset)
            body = offset + 12 + (name + 3) // 4 * 4
            if note == 32:
                meta = msgpack.unpackb(elf[body:body + desc], strict_map_key=False)
                return {q[".name"]: q for q in meta["amdhsa.kernels"]}
            step = body + (desc + 3) // 4 * 4 - offset
            offset, size = offset + step, size - step
    return {}


def test_evaluation_kernels_keep_the_box_in_registers():
    """Energies and forces of a batch read each replica's box into registers; a read of it at a computed place would put
    the whole of it into scratch memory."""
    k = {name: q for name, q in _kernels().items() if "6k_eval" in name}
    assert len(k) == 16   # two force types, forces and energies, single and batch, two pair styles
    held = {name: q[".private_segment_fixed_size"] for name, q in k.items()}
    assert max(held.values()) < BOX_BYTES, held
