"""What the built kernels ask of the device, read from the metadata of the library's own code objects."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1912_04791_amd", "libdsve.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libdsve.so not built")


def kernels():
    # the AMDGPU metadata notes (type 32): a header of three words, the name, a MessagePack map
    blob = open(LIB, "rb").read()
    found = {}
    for m in re.finditer(rb"AMDGPU\x00\x00", blob):
        name, size, kind = struct.unpack("<III", blob[m.start() - 12:m.start()])
        if (name, kind) == (7, 32):
            note = msgpack.unpackb(blob[m.end():m.end() + size], strict_map_key=False)
            found.update({k[".name"]: k for k in note["amdhsa.kernels"]})
    return found


def test_parts_hold_nothing_in_lds_but_what_they_exchange():
    # cells (3 doubles) and node terms (8, 5 or 6 words for FP64, mixed and the numerical eigensolver), and a
    # few words: an array per thread that the compiler puts there costs LDS and a read of host memory at the
    # start of every workgroup
    seen = 0
    for name, k in kernels().items():
        m = re.match(r"_ZN4dsve7k_partsILi(\d)ELi(\d)E", name)
        if not m:
            continue
        G, prec = map(int, m.groups())
        waves = 8 // (G + 1)
        exchanged = 8 * (3 * 63 * waves + G * (8, 5, 6)[prec] * 64 * waves)
        assert exchanged <= k[".group_segment_fixed_size"] <= exchanged + 256, name
        seen += 1
    assert seen >= 90


def test_parts_without_a_cut_carry_nothing_of_the_exchange():
    # k_parts<G, arithmetic, closure, cut>: fewer registers where no channel of the context is cut
    k = kernels()
    cut = [n for n in k if re.match(r"_ZN4dsve7k_partsILi\d(ELi\d){2}ELb1E", n)]
    assert len(cut) == 5 * 3 * 6
    for n in cut:
        assert k[n.replace("ELb1E", "ELb0E")][".vgpr_count"] < k[n][".vgpr_count"], n
