"""Rounding of the plane and cost kernels is written down, not left to the compiler: the front end's output allows no
contraction of a product and a sum anywhere in that file, so every instance of an evaluation rounds alike."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_operation_may_be_contracted(tmp_path):
    from paper_1805_07920_amd import build

    if not os.path.exists(build.hipcc()):
        pytest.skip("needs hipcc")
    out = tmp_path / "kernels.ll"
    subprocess.run([build.hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-w", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC,
                    "--offload-device-only", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes", "-o", str(out),
                    os.path.join(build.CSRC, "amh_kernels.hip")], check=True)
    functions = {m.group(1): m.group(0)
                 for m in re.finditer(r"^define [^@]*@(\S*3amh[^\s(]*)\((?:.|\n)*?^}", out.read_text(), re.M)}
    assert any("plane_q" in f for f in functions) and any("src_warp" in f for f in functions)
    assert not [f for f, body in functions.items() if re.search(r"= f(?:add|sub|mul) .*\bcontract\b", body)]
