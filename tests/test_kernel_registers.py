"""Registers and scratch memory of the built kernels, as the compiler wrote them beside the code: where they decide how many
workgroups share a compute unit, or whether a wavefront's data leaves the registers."""
import re
import struct

import msgpack
import pytest

from paper_2507_12205_amd import build


def kernels():
    """{(TM, DB, MODE, K, NB, VW): (VGPRs, scratch bytes per lane)} of the product kernel in the library."""
    data = open(build.LIB, "rb").read()
    base = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    (count,), pos, found = struct.unpack_from("<Q", data, base + 24), base + 32, {}
    for _ in range(count):
        offset, size, length = struct.unpack_from("<QQQ", data, pos)
        name = data[pos + 24:pos + 24 + length]
        pos += 24 + length
        if b"gfx950" not in name:
            continue
        elf = data[base + offset:base + offset + size]
        (shoff,) = struct.unpack_from("<Q", elf, 40)
        shentsize, shnum = struct.unpack_from("<HH", elf, 58)
        for i in range(shnum):
            kind, _, _, at, length = struct.unpack_from("<IQQQQ", elf, shoff + i * shentsize + 4)
            if kind != 7:                                            # notes
                continue
            namesz, descsz, note = struct.unpack_from("<III", elf, at)
            if note != 32:                                           # kernel metadata, in MessagePack
                continue
            start = at + 12 + (namesz + 3) // 4 * 4
            for k in msgpack.unpackb(elf[start:start + descsz], strict_map_key=False)["amdhsa.kernels"]:
                args = re.search(r"ecspmv_kernelI((?:Li\d+E){6})E", k[".name"])
                if args:
                    key = tuple(int(v) for v in re.findall(r"Li(\d+)E", args.group(1)))
                    found[key] = (k[".vgpr_count"], k[".private_segment_fixed_size"])
    return found


@pytest.fixture(scope="module")
def table():
    t = kernels()
    assert len(t) > 150 and {k[4] for k in t} == {1, 2, 4, 8} and {k[0] for k in t} == {0, 1, 3, 7, 15}
    return t


def test_no_scratch(table):
    # FP32 values with an 8- or 16-grained set: 32 and 64 value registers per unit, and no default build makes them
    spilling = {k: v for k, v in table.items() if v[1] and not (k[5] == 4 and k[0] >= 7)}
    assert not spilling, spilling


def test_two_workgroups_of_1024_threads(table):
    """64 VGPRs: 32 wavefronts on a compute unit.  One vector in FP16 with up to 4-grained sets, and several where LDS can
    hold two panels (launches in phases fill it)."""
    over = {k: v for k, v in table.items() if k[5] == 2 and k[2] != 3 and v[0] > 64
            and k[0] <= {1: 3, 2: 3, 4: 3, 8: 1}[k[4]]}
    assert not over, over
