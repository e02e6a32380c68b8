"""The projection dispatch on the CPU.

tests/host/gemm_dispatch_check.cpp compiles the projection source with its kernel
launches recorded and asks launch_gemm for every kind of product a forward has:
epilogue, rows, width, depth, weights as stored or as the fp16 image, device
width.  Every one is answered, and the kernels it chooses are exactly those that
the library holds: none is asked for that is not built, none is built that nothing
asks for.  And the products whose norm runs in the reduction do so where the test
of that kernel says."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

from paper_2608_28099_amd import build_lib

from . import test_gpu_reduce_norm as reduce_norm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host", "gemm_dispatch_check.cpp")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(SRC) and shutil.which("nm")),
                                reason="hipcc, nm or the check's source not available")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("dispatch")
    obj, exe = tmp / "check.o", tmp / "check"
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", SRC, "-o", str(obj)],
                   check=True, capture_output=True, text=True, timeout=300)
    subprocess.run([HIPCC, str(obj), "-o", str(exe)], check=True, capture_output=True, text=True, timeout=300)
    return str(exe)


def test_the_dispatch_reaches_what_is_built(check):
    res = subprocess.run([check], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    reached = set(res.stdout.split("\n")) - {""}
    if not os.path.exists(build_lib.LIB):
        build_lib.build()
    names = subprocess.run(["nm", "-C", build_lib.LIB], check=True, capture_output=True, text=True).stdout
    built = set(re.findall(r"__device_stub__(gemm_.*?)\(sp::", names))
    assert reached - built == set(), "chosen but not built"
    assert built - reached == set(), "built but never chosen"


@pytest.mark.parametrize("hidden,batch,intermediate,o,fc,down", reduce_norm.CASES)
def test_the_norm_runs_in_the_reduction(check, hidden, batch, intermediate, o, fc, down):
    """The products that test_gpu_reduce_norm.py is about are split as it says, and
    their norm is in the reduction."""
    qw = reduce_norm.HEADS * reduce_norm.HEAD_DIM
    widest = max(2 * intermediate, qw + 2 * reduce_norm.KV_HEADS * reduce_norm.HEAD_DIM, hidden)
    resid_row, resid_f32 = 1, 2
    for k, products in ((1, [(o, qw, resid_row)]), (2, [(fc, hidden, resid_f32), (o, qw, resid_f32),
                                                        (down, intermediate, resid_f32)])):
        part_bytes = 4 * max(16 * 32 * widest, 4 * min(batch * k, 1024) * hidden)
        for slices, depth, epi in products:
            out = subprocess.run([check, str(batch), str(hidden), str(depth), str(epi), str(part_bytes)], check=True,
                                 capture_output=True, text=True, timeout=60).stdout
            launches = [line.split("|") for line in out.strip().split("\n")]
            if slices == 1:
                assert len(launches) == 1 and launches[0][0].startswith("gemm_rows"), launches
            else:
                assert [x[0].split("<")[0] for x in launches] == ["gemm_lds", "gemm_reduce_norm"], launches
                assert int(launches[0][2]) == slices, launches
