"""Registers of the built kernels: a wavefront more or less per SIMD is not seen
in any result, so what the dispatch counts on is checked here."""
import re
import struct

import msgpack
import pytest

from paper_2008_11578_amd import orca


def _kernels():
    """Metadata of every kernel in the library, by mangled name (the notes of the
    gfx950 code objects inside it)."""
    blob = open(orca.LIB_PATH, "rb").read()
    found = {}
    for m in re.finditer(b"\x7fELF\x02\x01", blob):
        at = m.start()
        if struct.unpack_from("<H", blob, at + 18)[0] != 224:  # EM_AMDGPU
            continue
        phoff, = struct.unpack_from("<Q", blob, at + 32)
        phsize, phnum = struct.unpack_from("<HH", blob, at + 54)
        for k in range(phnum):
            head = at + phoff + k * phsize
            kind, = struct.unpack_from("<I", blob, head)
            if kind != 4:  # PT_NOTE
                continue
            off, = struct.unpack_from("<Q", blob, head + 8)
            size, = struct.unpack_from("<Q", blob, head + 32)
            p, end = at + off, at + off + size
            while p < end:
                namesz, descsz, typ = struct.unpack_from("<III", blob, p)
                desc = p + 12 + (namesz + 3) // 4 * 4
                if typ == 32:  # the kernels' metadata
                    for kern in msgpack.unpackb(blob[desc:desc + descsz])["amdhsa.kernels"]:
                        found[kern[".name"]] = kern
                p = desc + (descsz + 3) // 4 * 4
    return found


@pytest.fixture(scope="module")
def kernels():
    k = _kernels()
    assert len(k) > 50
    return k


@pytest.mark.parametrize("form,waves", [
    (r"6k_stepILi(4|8|10)ELi64ELb.ELb0", 4),
    (r"9k_adjointILi(4|8|10)ELi64ELb0ELb1", 4), (r"9k_adjointILi(4|8|10|12)ELi64ELb.ELb1", 3),
    (r"19k_step_batched_flatILi(4|8|10)ELi64", 3)])
def test_registers_leave_room_for_the_wavefronts_the_lds_does(kernels, form, waves):
    some = {n: k for n, k in kernels.items() if re.search(form, n)}
    assert some
    for n, k in some.items():
        # 512 registers of a SIMD lane, handed out by eights
        assert (k[".vgpr_count"] + 7) // 8 * 8 * waves <= 512, (n, k[".vgpr_count"])
        # a few registers of the steps with hard lines go to scratch memory
        hard = "6k_step" in n and "ELi64ELb1" in n
        assert k[".private_segment_fixed_size"] <= (96 if hard else 0), n
