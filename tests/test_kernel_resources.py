"""Registers of the built kernels, from the metadata of the code objects in
libmpstep.so (no GPU needed): the default kernels that must not spill."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2404_01035_amd", "libmpstep.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel name: (VGPRs spilled, bytes of scratch)}"""
    if not os.path.exists(LIB) or not os.path.exists(READELF) or not shutil.which("c++filt"):
        pytest.skip("library or binutils missing")
    co = str(tmp_path_factory.mktemp("co") / "k.co")
    data = open(LIB, "rb").read()
    out = {}
    at = data.find(MAGIC)
    while at >= 0:
        n, q = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n if n < 16 else 0):
            off, size, length = struct.unpack_from("<QQQ", data, q)
            name = data[q + 24:q + 24 + length]
            q += 24 + length
            if b"gfx950" in name:
                with open(co, "wb") as f:
                    f.write(data[at + off:at + off + size])
                notes = subprocess.run([READELF, "--notes", co], capture_output=True, text=True, check=True).stdout
                for m in re.finditer(r"- \.agpr_count:(.*?)\.wavefront_size", notes, re.S):
                    get = lambda key: re.search(r"\." + key + r":\s*(\S+)", m.group(1)).group(1)
                    out[get("name")] = (int(get("vgpr_spill_count")), int(get("private_segment_fixed_size")))
        at = data.find(MAGIC, at + 24)
    assert out, "no gfx950 kernels found"
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True).stdout.split("\n")
    return {n.split("(")[0].replace("void mp::", ""): v for n, v in zip(names, out.values())}


def test_3d_step_kernels_do_not_spill(kernels):
    steps = {n: v for n, v in kernels.items() if n.startswith(("k_step3d<", "k_step3d_gen<"))}
    assert len(steps) >= 32
    assert {n: v for n, v in steps.items() if v != (0, 0)} == {}
