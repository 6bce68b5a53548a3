"""What the compiler gave the kernels of the built library: registers spilled and
scratch memory, read from the metadata of its gfx950 code objects.

A spilled scalar register lives in a lane of a vector register, one move each way,
in the middle of the gather; a spilled vector register in scratch memory.  The
bounds are the counts from which a kernel was seen to lose time to them."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2504_07059_amd", "liblbm_mc.so")
BIN = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + 24)
        pos = at + 32
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", blob, pos)
            triple = blob[pos + 24:pos + 24 + tl].decode()
            pos += 24 + tl
            if "gfx950" in triple:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def _plain(mangled):
    """name<template arguments> of a mangled kernel name of the library."""
    m = re.match(r"_ZN5lbmmc(\d+)", mangled)
    if not m:
        return mangled
    at = m.end()
    name = mangled[at:at + int(m.group(1))]
    args = re.match(r"I((?:L[ib]\d+E)+)E", mangled[at + len(name):])
    if not args:
        return name
    return name + "<" + ", ".join(re.findall(r"L[ib](\d+)E", args.group(1))) + ">"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name<template arguments> of a kernel -> its resource counts."""
    if not os.path.exists(LIB) or not os.path.exists(os.path.join(BIN, "llvm-readelf")):
        pytest.skip("needs the built library and the ROCm binary tools")
    tmp = tmp_path_factory.mktemp("code_objects")
    out = {}
    for k, obj in enumerate(_code_objects(open(LIB, "rb").read())):
        path = str(tmp / f"{k}.elf")
        open(path, "wb").write(obj)
        notes = subprocess.run([os.path.join(BIN, "llvm-readelf"), "--notes", path],
                               capture_output=True, text=True, check=True).stdout
        for part in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", part).group(1)
            out[name] = {f: int(re.search(rf"\.{f}:\s+(\d+)", part).group(1))
                         for f in ("private_segment_fixed_size", "sgpr_spill_count",
                                   "vgpr_spill_count", "vgpr_count")}
    return {_plain(n): v for n, v in out.items()}


def _of(kernels, name):
    found = {k: v for k, v in kernels.items() if k.split("<")[0] == name}
    assert found, f"no kernel {name} in the library"
    return found


@pytest.mark.parametrize("name", ["k_step", "k_density", "k_moments", "k_adj_init"])
def test_kernels_with_every_species_in_a_thread(kernels, name):
    # a buffer resource per plane does not fit the scalar registers there: 519 to
    # 5207 of them spilled, and the equilibrium boundary ran at 0.4 to 0.6 of its speed
    bad = {k: v for k, v in _of(kernels, name).items()
           if v["sgpr_spill_count"] > 512 or v["private_segment_fixed_size"] > 0}
    assert not bad, bad


@pytest.mark.parametrize("args", ["0, 3, 2, true", "1, 2, 2, true", "1, 3, 2, true",
                                  "1, 4, 2, true", "1, 4, 16, false"])
def test_fused_reverse_pass_meets_the_waves_it_asks_for(tmp_path, args):
    # the compiler warns where a kernel's bound on waves per SIMD cannot be kept
    from paper_2504_07059_amd import build as B
    if not os.path.exists(B.HIPCC):
        pytest.skip("needs hipcc")
    src = tmp_path / "one.hip"
    src.write_text('#include "adjoint_impl.hpp"\nnamespace lbmmc {\n'
                   f"template __global__ void k_adj_fused<{args}>(const float*, const float*, "
                   "float*, const LatParams*, const Tile*, int, double*);\n}\n")
    r = subprocess.run([B.HIPCC] + B.FLAGS + ["--cuda-device-only", "-I" + B.CSRC, "-c",
                                              str(src), "-o", os.devnull],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert "failed to meet occupancy" not in r.stderr, r.stderr
