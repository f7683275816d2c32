"""Registers of the built kernels, read from the metadata of the library's
code objects (no GPU needed)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_15453_amd", "libstmoe.so")
LLVM = "/opt/rocm/llvm/bin"
READELF = os.path.join(LLVM, "llvm-readelf")
OBJCOPY = os.path.join(LLVM, "llvm-objcopy")


def _code_objects(tmp):
    fat = os.path.join(tmp, "fat")
    subprocess.run([OBJCOPY, f"--dump-section=.hip_fatbin={fat}", LIB, os.path.join(tmp, "copy.so")], check=True)
    data = open(fat, "rb").read()
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start()
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name without namespaces and arguments: (VGPRs, SGPRs)}"""
    tmp = str(tmp_path_factory.mktemp("co"))
    out = {}
    for i, co in enumerate(_code_objects(tmp)):
        path = os.path.join(tmp, f"{i}.co")
        with open(path, "wb") as f:
            f.write(co)
        notes = subprocess.run([READELF, "--notes", path], check=True, capture_output=True, text=True).stdout
        for k in re.split(r"\n  - ", notes):
            name = re.search(r"\.name:\s+(_Z\S+)", k)
            v, s = re.search(r"\.vgpr_count:\s+(\d+)", k), re.search(r"\.sgpr_count:\s+(\d+)", k)
            if name and v and s:
                d = subprocess.run(["c++filt", name.group(1)], check=True, capture_output=True, text=True).stdout
                d = re.sub(r"^void |stmoe::|\(anonymous namespace\)::", "", d.strip())
                out[re.sub(r"\(.*", "", d)] = (int(v.group(1)), int(s.group(1)))
    return out


def waves_per_simd(vgprs, sgprs):
    """512 VGPRs per lane in steps of 8 and 800 SGPRs in steps of 16 per SIMD, 8 waves at most."""
    up = lambda n, k: max(k, -(-n // k) * k)
    return min(8, 512 // up(vgprs, 8), 800 // up(sgprs, 16))


pytestmark = pytest.mark.skipif(
    not (os.path.exists(LIB) and os.path.exists(READELF) and os.path.exists(OBJCOPY) and shutil.which("c++filt")),
    reason="needs the built library and the ROCm binary utilities")


def test_routing_prologue_leaves_the_gemv_gate_up_its_waves(kernels):
    """The optional routing prologue of the GEMV gate/up kernels (up to two
    tokens) must not cost the calls that come with a selection a wave per
    SIMD: seven with the activations staged in LDS, eight without."""
    seen = 0
    for name, (v, s) in kernels.items():
        m = re.fullmatch(r"ffn_gate_up<(true|false), (16|32|64), 1, 2, (true|false)>", name)
        if m:
            seen += 1
            assert waves_per_simd(v, s) >= (7 if m.group(3) == "true" else 8), (name, v, s)
    assert seen == 12
