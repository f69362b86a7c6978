"""What the compiler gave the kernels of the built library, read from the metadata notes
of its gfx950 code objects.  No device."""
import os
import struct

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2203_07424_amd", "librec_mi355x.so")
SHT_NOTE, NT_AMDGPU_METADATA = 7, 32


def kernels(path):
    """{name: metadata} of every kernel in the 64-bit little-endian ELF files of the AMDGPU
    HSA ABI inside `path`."""
    with open(path, "rb") as f:
        data = f.read()
    found, at = {}, data.find(b"\x7fELF\x02\x01\x01\x40")
    while at >= 0:
        (table,), (entry, count) = struct.unpack_from("<Q", data, at + 0x28), struct.unpack_from("<HH", data, at + 0x3A)
        for i in range(count):
            _, kind, _, _, offset, size = struct.unpack_from("<IIQQQQ", data, at + table + i * entry)
            p, end = at + offset, at + offset + size
            while kind == SHT_NOTE and p < end:
                name_size, size_of_desc, note = struct.unpack_from("<III", data, p)
                desc = p + 12 + -(-name_size // 4) * 4
                if note == NT_AMDGPU_METADATA and data[p + 12:p + 18] == b"AMDGPU":
                    for k in msgpack.unpackb(data[desc:desc + size_of_desc])["amdhsa.kernels"]:
                        found[k[".name"]] = k
                p = desc + -(-size_of_desc // 4) * 4
        at = data.find(b"\x7fELF\x02\x01\x01\x40", at + 8)
    return found


@pytest.fixture(scope="module")
def built():
    from paper_2203_07424_amd import binding  # noqa: F401  (builds nothing, says so where the library is missing)
    ks = kernels(LIB)
    assert len(ks) > 100 and any("fc_big_behind_scan_kernel" in n for n in ks)
    return ks


def test_no_kernel_has_scratch_memory(built):
    """The library allocates no device memory; scratch would be the runtime's, behind its back."""
    assert {n: k[".private_segment_fixed_size"] for n, k in built.items() if k[".private_segment_fixed_size"]} == {}
