"""Registers of kernels whose launches have more workgroups than one wave a SIMD needs, read from the built library: as many waves a SIMD as
their launches were measured with."""
import os
import re
import struct
import subprocess

import pytest

from paper_2006_13486_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"

# template arguments of spmm_reg (stage, rows a tile row, tap-grouped, groups, column tiles, one register set, stage of the layout, two
# chains), spmm_reg_bf16 (stage, rows a tile row, groups, columns, one register set, stage of the layout, two chains), sddmm_reg and sddmm_lines (row groups, step groups,
# bf16, convolution, all of G_i[, 64-bit offsets]) -> waves a SIMD.  sddmm_lines has two waves a SIMD in a workgroup: four are two of those.
WAVES = {f"spmm_reg_bf16<36, {rs}, 1, 64, 0, 36, 0>": 4 for rs in (2, 4, 8, 16)}
WAVES.update({f"spmm_reg_bf16<8, {rs}, 1, 64, 0, 8, 0>": 7 for rs in (2, 4, 8, 16)})
WAVES.update({f"spmm_reg_bf16<8, {rs}, 2, 64, 0, 8, 0>": 4 for rs in (2, 4, 8, 16)})
WAVES.update({"spmm_reg<32, 16, 0, 1, 0, 1, 32, 0>": 4, "spmm_reg<36, 16, 1, 1, 0, 1, 36, 0>": 4, "spmm_reg<72, 16, 1, 1, 0, 1, 72, 0>": 4})
WAVES.update({f"sddmm_reg<2, 2, {b}, 0, 1>": 4 for b in (0, 1)})
WAVES.update({"sddmm_reg<1, 1, 0, 0, 1>": 8})
WAVES.update({f"sddmm_lines<2, 1, 1, 1, {g}, 1>": 4 for g in (0, 1)})


def _code_objects(path):
    """The GPU code objects in a host library: entries of its __CLANG_OFFLOAD_BUNDLE__ containers."""
    blob = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(magic, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not (os.path.exists(build.LIB) and os.path.exists(READELF)):
        pytest.skip("needs the built library and llvm-readelf")
    d = tmp_path_factory.mktemp("code")
    found = {}
    for k, obj in enumerate(_code_objects(build.LIB)):
        f = d / f"{k}.co"
        f.write_bytes(obj)
        text = subprocess.check_output([READELF, "--notes", str(f)], text=True)
        for part in text.split("- .agpr_count:")[1:]:
            get = lambda key: re.search(rf"\.{key}:\s+(\S+)", part)[1]
            found[get("name").strip("'")] = (int(get("vgpr_count")), int(get("vgpr_spill_count")))
    names = list(found)
    plain = subprocess.check_output(["c++filt"], input="\n".join(names), text=True).splitlines()
    short = lambda s: re.sub(r"\(anonymous namespace\)::|^void ", "", s).replace("true", "1").replace("false", "0")
    return {short(p): found[n] for n, p in zip(names, plain)}


@pytest.mark.parametrize("prefix", WAVES)
def test_waves_a_simd(kernels, prefix):
    some = {name: regs for name, regs in kernels.items() if name.startswith(prefix)}
    assert some, sorted(kernels)[:5]
    for name, (registers, spilled) in some.items():
        # (512 registers a lane and SIMD, of both kinds, given out in eights; at most eight waves)
        waves = min(8, 512 // ((registers + 7) // 8 * 8))
        assert waves >= WAVES[prefix] and spilled == 0, (name, registers, spilled)
