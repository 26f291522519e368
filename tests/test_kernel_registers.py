"""Vector registers of the built tile forwards, read from the code objects in the library: up to 16
states five waves must fit a SIMD (96 of its 512 registers each), or the grid of a batch under many
models holds too few workgroups for each."""
import struct

import msgpack
import pytest

from paper_1310_3322_amd import hmm

NT_AMDGPU_METADATA = 32


def kernels():
    """Metadata of every kernel of the library, by mangled name."""
    data = open(hmm.LIB_PATH, "rb").read()
    out = {}
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:  # EM_AMDGPU
            phoff, = struct.unpack_from("<Q", data, at + 32)
            phentsize, phnum = struct.unpack_from("<HH", data, at + 54)
            for p in range(phnum):
                kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", data, at + phoff + p * phentsize)
                n, end = at + off, at + off + size
                while kind == 4 and n < end:  # PT_NOTE
                    namesz, descsz, ntype = struct.unpack_from("<III", data, n)
                    desc = n + 12 + (namesz + 3) // 4 * 4
                    if ntype == NT_AMDGPU_METADATA:
                        for k in msgpack.unpackb(data[desc:desc + descsz])["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    n = desc + (descsz + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 1)
    return out


@pytest.mark.parametrize("name,registers", [("k_fwd_mfmaILi1ELb1ELb0E", 96), ("k_fwd_mfmaILi1ELb0ELb0E", 96),
                                            ("k_fwd_mfma32ILi1ELb1E", 128), ("k_fwd_mfma32ILi1ELb0E", 128)])
def test_waves_per_simd(name, registers):
    found = [k for n, k in kernels().items() if name in n]
    assert len(found) == 1
    assert found[0][".vgpr_count"] + found[0].get(".agpr_count", 0) <= registers
