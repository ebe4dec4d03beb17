"""How launches are split, on the CPU.  The scratch by which tp_slice_forward_static admits a slice covers the split plan
that its kernels then follow, and an admitted plan stays within the static array: every
forward product of widths 64 to 16384 and slices of 1 to 4096 rows, in bf16 and fp32,
planned and "launched" on the CPU by tests/native/plan_driver.cpp, whose stand-ins for
the HIP runtime record what a launch is given.  The same driver checks the least work
of a part of a split column sum or dQ launch (256 rows or keys).  Which slices are admitted is pinned by
a table of answers."""
import os
import subprocess

import pytest

from paper_2102_07988_amd import terapipe as tp
from paper_2102_07988_amd.build import HIPCC
from test_abi import _init

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBDIR = os.path.join(ROOT, "paper_2102_07988_amd", "lib")


def test_admission_covers_the_plan_that_runs(tmp_path):
    exe = str(tmp_path / "plan_driver")
    obj = str(tmp_path / "plan_driver.o")
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-w", "-x", "hip", "-c",
                    os.path.join(ROOT, "tests", "native", "plan_driver.cpp"), "-o", obj],
                   check=True)
    subprocess.run([HIPCC, "-rdynamic", obj, "-o", exe, os.path.join(LIBDIR, "libterapipe.so"),
                    "-Wl,-rpath," + LIBDIR], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-2000:]
    assert "products" in r.stdout


LENS = (1, 16, 64, 100, 128, 144, 200, 256, 257, 400, 512, 777, 1024, 2048, 4096)


@pytest.mark.parametrize("H,d,parts,dtype,batch,refused", [
    (2048, 128, 1, "bf16", 1, (257, 777)),
    (5120, 128, 1, "bf16", 1, (100, 144, 200, 256, 257, 400, 512, 777, 1024, 2048, 4096)),
    (12288, 128, 1, "bf16", 1, (100, 128, 144, 200, 256, 257, 400, 512, 777, 2048)),
    (12288, 128, 8, "bf16", 1, (100, 200, 256, 257, 400, 512, 777, 1024, 2048, 4096)),
    (2048, 64, 1, "bf16", 3, (100, 257, 512, 777, 1024)),
    (1536, 32, 1, "bf16", 1, (777, 2048, 4096)),
    (4096, 64, 1, "fp32", 1, ()),
])
def test_which_slices_are_admitted(H, d, parts, dtype, batch, refused):
    """The admission is checked before the order, so an admitted slice of a stage
    without a sequence answers TP_ERR_ORDER."""
    for n in LENS:
        rc, h = _init(tp.make_config(1, H, H // d, n, dtype, batch=batch, op_parts=parts))
        assert rc == tp.TP_OK
        s = tp.lib.tp_slice_forward_static(h, 0, n, 0x7e0000000000, 0x7d0000000000)
        assert s == (tp.TP_ERR_WORKSPACE if n in refused else tp.TP_ERR_ORDER), n
        tp.lib.tp_stage_destroy(h)
