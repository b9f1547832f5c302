"""Registers of the built kernels, from the metadata of the library's gfx950 code object (no GPU)."""
import os
import re
import struct

import msgpack
import pytest

from paper_2412_07894_amd import binding, build


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    data = open(binding.LIB_PATH, "rb").read()
    base = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    n, at = struct.unpack_from("<Q", data, base + 24)[0], base + 32
    for _ in range(n):
        off, size, tl = struct.unpack_from("<QQQ", data, at)
        if data[at + 24:at + 24 + tl].endswith(b"gfx950"):
            elf = data[base + off:base + off + size]
        at += 24 + tl
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3a)
    found = {}
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        if kind != 7:                            # SHT_NOTE
            continue
        at, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        end = at + size
        while at < end:
            namesz, descsz, typ = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if typ == 32 and elf[at + 12:at + 18] == b"AMDGPU":
                for k in msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]:
                    found[k[".name"]] = k
            at = desc + (descsz + 3) // 4 * 4
    return found


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("split", [0, 1])
def test_own_items_keep_one_set_of_accumulators(kernels, d, split):
    """The own-item forward runs the tile loop of the listed one.  Where the compiler knows the item to be the workgroup's it makes
    scalar branches of the diagonal's mask, keeps the accumulators twice and copies them in every tile, which shows
    in the registers: 38 more."""
    name = {own: [n for n in kernels if re.search(rf"hyd_fwd_bf16_kernelILb0ELi{d}ELi{split}E", n) and ("SelfSchedule" in n) == own] for own in (False, True)}
    assert len(name[False]) == len(name[True]) == 1
    listed, own = (kernels[name[x][0]] for x in (False, True))
    assert own[".vgpr_count"] <= listed[".vgpr_count"]
    assert own[".vgpr_spill_count"] == 0 and own[".private_segment_fixed_size"] == 0
