"""Kernels on the main path of batches that must keep their registers: one that spills
writes its scratch memory in every launch, whatever the launch's size."""
import os
import struct

import pytest

from paper_2512_23314_amd import _build


def _scratch(lib):
    """Scratch bytes per lane of each kernel in the library, from the notes of its
    code objects (note name "AMDGPU", type 32: a msgpack map)."""
    msgpack = pytest.importorskip("msgpack")
    data = open(lib, "rb").read()
    out, at = {}, data.find(b"AMDGPU\0\0")
    while at >= 0:
        namesz, descsz, kind = struct.unpack_from("<III", data, at - 12)
        if namesz == 7 and kind == 32:
            for k in msgpack.unpackb(data[at + 8:at + 8 + descsz])["amdhsa.kernels"]:
                out[k[".name"]] = k[".private_segment_fixed_size"]
        at = data.find(b"AMDGPU\0\0", at + 8)
    return out


@pytest.mark.skipif(not os.path.exists(_build.LIB), reason="the library is not built")
def test_batch_scan_keeps_its_registers():
    scratch = _scratch(_build.LIB)
    # instances <ODD, LEAN, SEGT>: with and without a short final key, dense hashes
    for args in ("Lb1ELb0ELb0E", "Lb0ELb0ELb0E", "Lb0ELb0ELb1E", "Lb0ELb1ELb0E"):
        names = [n for n in scratch if "k_probe_textI" + args in n]
        assert len(names) == 1, sorted(scratch)
        assert scratch[names[0]] == 0, names[0]
