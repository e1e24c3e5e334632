"""Register spills of the built kernels, read from the metadata in the library
(the code objects of its fat binary): the kernels of the reverse sweep's large
levels keep their values in registers.  Scratch traffic in the inner loops cost
one undetected mode of cutoff 20 behind seven detected ones of cutoff 3 a third
of its reverse sweep's time."""
import os
import re
import struct

import msgpack
import pytest

from paper_2303_08879_amd import fockdiag as F

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, ids = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + ids]
            p += 24 + ids
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, p)


def kernels(elf):
    """The kernels' metadata (the AMDGPU note, msgpack) of one code object."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, num = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(num):
        typ, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        off, length = struct.unpack_from("<QQ", elf, shoff + i * size + 0x18)
        if typ != 7:   # SHT_NOTE
            continue
        p = off
        while p < off + length:
            nl, dl, kind = struct.unpack_from("<III", elf, p)
            name = elf[p + 12:p + 12 + nl].rstrip(b"\0")
            d = p + 12 + (nl + 3) // 4 * 4
            if name == b"AMDGPU" and kind == 32:
                yield from msgpack.unpackb(elf[d:d + dl], strict_map_key=False)["amdhsa.kernels"]
            p = d + (dl + 3) // 4 * 4


@pytest.fixture(scope="module")
def spills():
    if not os.path.exists(F.LIB_PATH):
        pytest.skip("the library is not built")
    out = {}
    for elf in code_objects(open(F.LIB_PATH, "rb").read()):
        for k in kernels(elf):
            out[k[".name"]] = k[".vgpr_spill_count"]
    assert len(out) > 100
    return out


def test_reverse_block_kernels_do_not_spill(spills):
    # k_vjp_block<detected modes, block coordinates, precision, streamed rows>:
    # with rows in LDS nothing spills in double precision (but for 7 registers of
    # <5, 4>, whose build without is 10 % slower); in single precision only past 16
    # positions, where two wavefronts with spills beat one without
    seen, bad = 0, []
    for name, n in spills.items():
        m = re.match(r"_ZN2fd11k_vjp_blockILi(\d)ELi(\d)E([df])Lb0EE", name)
        if not m:
            continue
        seen += 1
        md, nq, r = int(m[1]), int(m[2]), m[3]
        if n > (8 if (md, nq, r) == (5, 4, "d") else 0 if r == "d" or nq + 2 * md < 16 else 4 if nq + 2 * md == 16 else 128):
            bad.append((md, nq, r, n))
    assert seen == 2 * 8 * 3
    assert not bad


@pytest.mark.parametrize("kernel", ["k_vjp_point", "k_fwd_point", "k_state_vjp", "k_point_small_vjp"])
def test_point_kernels_do_not_spill(spills, kernel):
    mine = {k: n for k, n in spills.items() if re.match(rf"_ZN2fd{len(kernel)}{kernel}I", k)}
    assert mine and not any(mine.values()), {k: n for k, n in mine.items() if n}
