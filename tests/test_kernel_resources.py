"""What the compiler made of the kernels, from the metadata of the library that was built here: kernels whose loops hold their sums in
registers keep them there."""
import os
import struct

import msgpack
import pytest

import paper_1412_6249_amd as pa

LIB = os.path.join(os.path.dirname(pa.__file__), "libpurine_conv.so")


def _code_objects(blob):
    """The GPU code objects of a library: whole ELF files inside its fat binary (e_machine 224)."""
    at = blob.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:
            yield at
        at = blob.find(b"\x7fELF", at + 4)


def _metadata(blob, elf):
    """The AMDGPU metadata notes (name "AMDGPU", type 32: one msgpack document) of the code object at `elf`."""
    shoff, shentsize, shnum = struct.unpack_from("<Q", blob, elf + 40)[0], *struct.unpack_from("<HH", blob, elf + 58)
    for i in range(shnum):
        kind, offset, size = struct.unpack_from("<I", blob, elf + shoff + i * shentsize + 4)[0], *struct.unpack_from("<QQ", blob, elf + shoff + i * shentsize + 24)
        end, p = elf + offset + size, elf + offset
        while kind == 7 and p < end:
            namesz, descsz, what = struct.unpack_from("<III", blob, p)
            desc = p + 12 + (namesz + 3) // 4 * 4
            if what == 32 and blob[p + 12:p + 18] == b"AMDGPU":
                yield msgpack.unpackb(blob[desc:desc + descsz])
            p = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    blob = open(LIB, "rb").read()
    found = {k[".name"]: k for elf in _code_objects(blob) for doc in _metadata(blob, elf) for k in doc["amdhsa.kernels"]}
    assert len(found) > 100
    return found


@pytest.mark.parametrize("name", ["wgrad_staged_kernel", "conv_direct_kernel", "fc_direct_kernel", "wgrad_reduce"])
def test_no_register_goes_to_memory(kernels, name):
    mine = {n: k for n, k in kernels.items() if name in n}
    assert mine
    bad = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in mine.items()
           if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not bad, bad
