"""The projection dispatch on the CPU.

tests/host/gemm_dispatch_check.cpp compiles the projection source with its kernel
launches recorded and asks launch_gemm for every kind of product a forward has:
epilogue, rows, width, depth, weights as stored or as the fp16 image, device
width.  Every one is answered, and the kernels it chooses are exactly those that
the library holds: none is asked for that is not built, none is built that nothing
asks for."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

from paper_2608_28099_amd import build_lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host", "gemm_dispatch_check.cpp")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(SRC) and shutil.which("nm")),
                    reason="hipcc, nm or the check's source not available")
def test_the_dispatch_reaches_what_is_built(tmp_path):
    obj, exe = tmp_path / "check.o", tmp_path / "check"
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", SRC, "-o", str(obj)],
                   check=True, capture_output=True, text=True, timeout=300)
    subprocess.run([HIPCC, str(obj), "-o", str(exe)], check=True, capture_output=True, text=True, timeout=300)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    reached = set(res.stdout.split("\n")) - {""}
    if not os.path.exists(build_lib.LIB):
        build_lib.build()
    names = subprocess.run(["nm", "-C", build_lib.LIB], check=True, capture_output=True, text=True).stdout
    built = set(re.findall(r"__device_stub__(gemm_.*?)\(sp::", names))
    assert reached - built == set(), "chosen but not built"
    assert built - reached == set(), "built but never chosen"
