"""Registers of the built kernels, read from the code objects in the library: a
kernel that needs more loses waves per SIMD, which no result shows."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

from paper_1109_2935_amd import build

EM_AMDGPU = 224
NT_AMDGPU_METADATA = 32


def code_objects(data):
    """The gfx950 ELF images embedded in a shared library."""
    at = data.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            yield at
        at = data.find(b"\x7fELF", at + 4)


def kernels(path):
    """{mangled name: metadata} of every kernel in the library."""
    data, out = open(path, "rb").read(), {}
    for at in code_objects(data):
        phoff, phsize, phnum = (struct.unpack_from(f, data, at + o)[0] for f, o in (("<Q", 32), ("<H", 54), ("<H", 56)))
        for i in range(phnum):
            kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", data, at + phoff + i * phsize)
            if kind != 4:  # PT_NOTE
                continue
            p, end = at + offset, at + offset + size
            while p < end:
                nname, ndesc, ntype = struct.unpack_from("<III", data, p)
                desc = p + 12 + (nname + 3) // 4 * 4
                if ntype == NT_AMDGPU_METADATA:
                    for k in msgpack.unpackb(data[desc:desc + ndesc], raw=False).get("amdhsa.kernels", ()):
                        out[k[".name"]] = k
                p = desc + (ndesc + 3) // 4 * 4
    return out


@pytest.fixture(scope="module")
def table():
    if not os.path.exists(build.OUT):
        pytest.skip("the library is not built")
    return kernels(build.OUT)


# A SIMD has 512 vector registers per lane, given out in eights: 168 for three
# waves. The second half of the Schur operator (mode 2, with and without partial
# sums) is bound by memory latency, and fell from 100 to 111 us with two (BF16, 18
# reals, 32^3 x 64).
@pytest.mark.parametrize("storage", ["DF16_", "NS_4bf16E"])
@pytest.mark.parametrize("recon", [12, 18])
@pytest.mark.parametrize("partials", [0, 1])
def test_schur_second_half_keeps_three_waves(table, storage, recon, partials):
    name = "_ZN4lqcd13wilson_kernelI%sfLi%dELi2ELb%dELi1EEEvNS_5WArgsIT_EE" % (storage, recon, partials)
    k = table[name]
    assert k[".vgpr_count"] <= 168 and k[".private_segment_fixed_size"] == 0, k
