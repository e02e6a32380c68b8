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

from . import test_gpu_gemm_stream as gemm_stream
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


@pytest.mark.parametrize("intermediate,batch,tile", gemm_stream.CASES)
def test_streaming_tiles_run_where_their_test_says(check, intermediate, batch, tile):
    hidden, qw = gemm_stream.HIDDEN, gemm_stream.HEADS * gemm_stream.HEAD_DIM
    part_bytes = 4 * max(16 * 32 * 2 * intermediate, 4 * batch * hidden)

    def streaming(width, depth, epi):  # the tile that a product runs on, if a streaming one
        out = subprocess.run([check, str(batch), str(width), str(depth), str(epi), str(part_bytes)], check=True,
                             capture_output=True, text=True, timeout=60).stdout
        m = re.match(r"gemm_lds<(\d+), (\d+), \d+, \d+, \d+, 64, true,", out)
        return f"{m[1]}x{m[2]}" if m else None

    assert streaming(2 * intermediate, hidden, SWIGLU) == tile
    if batch > 16:  # o and down
        assert streaming(hidden, qw, RESID_ROW) and streaming(hidden, intermediate, RESID_F32)


STORE, RESID_ROW, RESID_F32, SWIGLU = 0, 1, 2, 3
# rows, width, depth, epilogue; us of plans (tile / K slices, or the row kernel), fp16
# image.  Off the heads the streaming tiles were tuned on, then on them
MEASURED = [
    (65, 16384, 3072, SWIGLU, {"128x64/1": 23.1, "128x96/1": 29.7, "64x64/1": 30.1}),
    (33, 16384, 1024, SWIGLU, {"64x64/1": 9.2, "128x64/1": 9.4, "64x96/1": 11.3}),
    (17, 1536, 6144, SWIGLU, {"32x128/8": 10.9, "rows": 18.2}),
    (12, 9728, 3072, SWIGLU, {"16x32/1": 14.8, "16x96/1": 18.2, "rows": 20.2}),
    (128, 3072, 1024, STORE, {"16x32/1": 6.6, "64x64/1": 6.9, "128x64/4": 11.4}),
    (33, 2048, 1024, STORE, {"16x16/1": 5.0, "rows": 5.2, "64x64/4": 8.1}),
    (64, 24576, 4096, SWIGLU, {"64x96/1": 34.8, "64x160/1": 43.3, "128x64/1": 53.3}),
    (128, 5120, 17408, RESID_F32, {"128x160/8": 44.4, "128x128/6": 47.0, "256x128/6": 49.6}),
    (16, 4096, 12288, RESID_F32, {"16x64/4": 23.7, "rows": 27.2}),
]


@pytest.mark.parametrize("rows,width,depth,epi,times", MEASURED)
def test_the_chosen_plan_is_near_the_fastest(check, rows, width, depth, epi, times):
    out = subprocess.run([check, str(rows), str(width), str(depth), str(epi), str(1 << 28)], check=True,
                         capture_output=True, text=True, timeout=60).stdout
    kernel, _, slices, _ = out.strip().split("\n")[0].split("|")
    tile = re.match(r"gemm_lds<(\d+), (\d+),", kernel)
    plan = f"{tile[1]}x{tile[2]}/{slices}" if tile else "rows"
    assert plan in times, plan
    assert times[plan] <= 1.15 * min(times.values()), plan
