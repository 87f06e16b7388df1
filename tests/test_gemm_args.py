"""The projections' launcher refuses operands in different layouts
(tests/native/gemm_args.hip, host code linked with the built library; the
refused calls launch nothing, so it needs no GPU and is not run on one)."""

import os
import shutil
import subprocess

import pytest
import torch

from paper_2607_18839_amd import build

TESTS = os.path.dirname(os.path.abspath(__file__))

pytestmark = [pytest.mark.skipif(not shutil.which(build.HIPCC), reason="hipcc not available"),
              pytest.mark.skipif(torch.cuda.is_available(), reason="host check")]


def test_mixed_layouts_are_refused(tmp_path):
    exe = str(tmp_path / "gemm_args")
    r = subprocess.run([build.HIPCC, "-std=c++17", "-O1", "--cuda-host-only", "-I" + os.path.join(build.ROOT, "include"),
                        "-I" + build.CSRC, os.path.join(TESTS, "native", "gemm_args.hip"), "-L" + build.PKG, "-lhpd",
                        "-Wl,-rpath," + build.PKG, "-o", exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
