"""What the built kernels take of a compute unit, read from the metadata of the library's code object."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2007_16100_amd import spv

AMDGPU, NOTE, METADATA = 224, 7, 32  # e_machine, section type, note type


def kernels():
    """{demangled name: metadata} of every kernel in the library."""
    data, found, at = open(spv.LIB_PATH, "rb").read(), {}, 0
    while (at := data.find(b"\x7fELF\x02\x01\x01", at)) >= 0:
        base, at = at, at + 4
        if struct.unpack_from("<H", data, base + 18)[0] != AMDGPU:
            continue
        table, = struct.unpack_from("<Q", data, base + 40)
        size, count = struct.unpack_from("<HH", data, base + 58)
        for i in range(count):
            head = base + table + i * size
            if struct.unpack_from("<I", data, head + 4)[0] != NOTE:
                continue
            off, left = struct.unpack_from("<QQ", data, head + 24)
            p, end = base + off, base + off + left
            while p < end:
                name, desc, kind = struct.unpack_from("<III", data, p)
                p += 12 + (name + 3) // 4 * 4
                if kind == METADATA:
                    for k in msgpack.unpackb(data[p:p + desc])["amdhsa.kernels"]:
                        found[k[".name"]] = k
                p += (desc + 3) // 4 * 4
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout
    return dict(zip(names.split("\n"), found.values()))


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(spv.LIB_PATH):
        pytest.skip("libspv.so is not built")
    return kernels()


def test_neighbour_table_kernels_keep_their_registers(built):
    """Every tile of the neighbour-table convs, on 27 and on 8 offsets, holds its rows, sums and fragments in
    registers (512 per lane and SIMD, shared by the waves of the workgroups that its rule counts on per CU)."""
    union = {n: k for n, k in built.items() if "k_conv_union<" in n}
    per_k3 = {k3: sum(re.search(r"k_conv_union<\d+, %d," % k3, n) is not None for n in union) for k3 in (27, 8)}
    assert per_k3[27] > 0 and per_k3[8] > 0
    spilled = [n for n, k in union.items() if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]]
    assert not spilled, spilled
