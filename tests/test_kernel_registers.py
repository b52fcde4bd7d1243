"""What the compiler made of kernels whose registers are just enough, read from the metadata of the built library: the number of
spilled vector registers of an instantiation is stated beside its code, and a change that brings them back goes unnoticed otherwise."""
import os
import struct

import pytest

from paper_2403_20137_amd import kvbfp

msgpack = pytest.importorskip("msgpack")
EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def kernels():
    """{mangled name: metadata} of all code objects in libkvbfp.so."""
    data, found, at = open(kvbfp.LIB_PATH, "rb").read(), {}, 0
    while (at := data.find(b"\x7fELF\x02\x01", at + 4)) >= 0:
        machine, = struct.unpack_from("<H", data, at + 18)
        if machine != EM_AMDGPU:
            continue
        shoff, = struct.unpack_from("<Q", data, at + 40)
        shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
        for i in range(shnum):
            kind, = struct.unpack_from("<I", data, at + shoff + i * shentsize + 4)
            if kind != SHT_NOTE:
                continue
            off, size = struct.unpack_from("<QQ", data, at + shoff + i * shentsize + 24)
            pos = at + off
            while pos < at + off + size:
                namesz, descsz, note = struct.unpack_from("<III", data, pos)
                desc = pos + 12 + (namesz + 3) // 4 * 4
                if note == NT_AMDGPU_METADATA:
                    for k in msgpack.unpackb(data[desc:desc + descsz])["amdhsa.kernels"]:
                        found[k[".name"]] = k
                pos = desc + (descsz + 3) // 4 * 4
    return found


@pytest.mark.skipif(not os.path.exists(kvbfp.LIB_PATH), reason="library not built")
def test_fp32_pass_for_five_to_eight_heads_has_no_spills():
    # decode_split_mfma_p4<N, HG = 2, PL = 3, PAGED, SHARE, THREE = false>: 16 instantiations
    got = {n: k[".vgpr_spill_count"] for n, k in kernels().items() if "decode_split_mfma_p4I" in n and "ELi2ELi3E" in n}
    assert len(got) == 16 and not any(got.values()), got
