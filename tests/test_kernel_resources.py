"""Registers and scratch of the compiled sweeps: a step's coefficients belong in
scalar registers, which leaves the vector registers to the planes in flight."""
import os
import re
import struct
import subprocess

import pytest

from paper_0911_5692_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 code objects in a library's offload bundles."""
    at = data.find(BUNDLE)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + ln]:
                yield data[at + off:at + off + size]
            p += 24 + ln
        at = data.find(BUNDLE, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        data = f.read()
    out, tmp = {}, tmp_path_factory.mktemp("co") / "x.co"
    for co in _code_objects(data):
        tmp.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(tmp)], capture_output=True, text=True, check=True).stdout
        for k in re.split(r"\n  - \.agpr_count:", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", k).group(1)
            m = re.search(r"k_sweep_lds(27)?I([fd])Li(\d)ELi(\d+)ELi(\d+)E", name)
            if m:
                num = {a: int(re.search(r"\.%s:\s+(\d+)" % a, k).group(1))
                       for a in ("vgpr_count", "private_segment_fixed_size")}
                key = (27 if m.group(1) else 7, {"f": "f32", "d": "f64"}[m.group(2)],
                       int(m.group(4)), int(m.group(5)), int(m.group(3)))
                out[key] = num
    return out


# scratch bytes a lane, most over beta 2 to 6, next to none of it touched in the
# loop over planes; every other tile has none
SCRATCH = {(7, "f32", 64, 16): 32, (7, "f64", 32, 16): 16, (27, "f32", 64, 8): 16, (27, "f32", 128, 4): 36,
           (27, "f32", 64, 16): 24, (27, "f32", 128, 8): 24, (27, "f64", 128, 4): 24}


@pytest.mark.parametrize("stencil,tiles", [(7, [(32, 8), (32, 16), (64, 4), (64, 8), (64, 16), (128, 4), (128, 8)]),
                                           (27, [(64, 4), (64, 8), (64, 16), (128, 4), (128, 8)])])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_scratch(kernels, stencil, tiles, dtype):
    for tx, ty in tiles:
        for nh in range(1, 6):
            k = kernels[stencil, dtype, tx, ty, nh]
            assert k["private_segment_fixed_size"] <= SCRATCH.get((stencil, dtype, tx, ty), 0), (tx, ty, nh)


def test_registers(kernels):
    """Waves per SIMD of the tiles that fill the device with few registers: 512
    registers a lane, in steps of 8."""
    for nh in range(1, 6):
        assert kernels[7, "f64", 64, 8, nh]["vgpr_count"] <= 168  # three
        assert kernels[7, "f32", 32, 16, nh]["vgpr_count"] <= 96  # five
