"""Compiles and runs a C++ main() against the library's headers on the CPU."""
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
needs_hipcc = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")


def run(source: str) -> str:
    """The program's output; its exit status must be 0."""
    with tempfile.TemporaryDirectory() as d:
        src, exe = os.path.join(d, "unit.hip"), os.path.join(d, "unit")
        with open(src, "w") as f:
            f.write(source)
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-std=c++17", "-O1", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_1709_03565_amd", "csrc"), "-o", exe, src],
                       check=True, capture_output=True)
        return subprocess.run([exe], capture_output=True, text=True, check=True, timeout=60).stdout
