"""Registers and scratch of the kernels as they were compiled, from the metadata the compiler left in the library."""
import struct

import msgpack
import pytest

from paper_2012_15667_amd import binding as B

EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def _kernels():
    """{mangled name: metadata} of every gfx950 kernel in the built library."""
    data = open(B.LIB_PATH, "rb").read()
    found, at = {}, data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            table, = struct.unpack_from("<Q", data, at + 40)
            size, count = struct.unpack_from("<HH", data, at + 58)
            for i in range(count):
                _, kind, _, _, offset, length = struct.unpack_from("<IIQQQQ", data, at + table + i * size)
                if kind != SHT_NOTE:
                    continue
                p, end = at + offset, at + offset + length
                while p < end:
                    name, desc, what = struct.unpack_from("<III", data, p)
                    p += 12 + (name + 3) // 4 * 4
                    if what == NT_AMDGPU_METADATA:
                        for k in msgpack.unpackb(data[p:p + desc])["amdhsa.kernels"]:
                            found[k[".name"]] = k
                    p += (desc + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)
    return found


@pytest.fixture(scope="module")
def kernels():
    k = _kernels()
    assert len(k) > 100
    return k


@pytest.mark.parametrize("m", [2, 3, 4, 6])
@pytest.mark.parametrize("vec", [0, 1])
def test_kernels_parts_do_not_cost_the_input_transform_its_waves(kernels, m, vec):
    """Kernels are cut into parts and inputs transformed in one launch: cutting must not take more registers than leave a SIMD as
    many waves as the launch without it has (512 registers a lane, in steps of eight)."""
    waves = {}
    for kind in (0, 1, 2):                                   # plain kernels, parts from w, parts from a caller's U
        names = [k for k in kernels if "10transformsILi%dELb%dELi%dE" % (m, vec, kind) in k]
        assert len(names) == (0 if m in (3, 6) and vec else 1), (kind, names)
        for n in names:
            waves[kind] = min(8, 512 // (-(-kernels[n][".vgpr_count"] // 8) * 8))
    if waves:
        assert waves[1] >= min(waves[0], waves[2]), waves
