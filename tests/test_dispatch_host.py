"""Every kind of matrix product starts a kernel for the tile configurations it has and refuses all others."""
import os
import shutil
import subprocess

import pytest

from paper_2002_02885_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_product_without_a_kernel_for_its_tiles_is_refused(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc to compile the driver with")
    binding.lib()
    exe = str(tmp_path / "dispatch")
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-I", build.CSRC, os.path.join(ROOT, "tests", "dispatch_driver.cpp"),
                    "-o", exe, "-Xlinker", build.LIB, "-Xlinker", "-rpath=" + os.path.dirname(build.LIB)], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100, env={**os.environ, "HIP_VISIBLE_DEVICES": "-1", "ROCR_VISIBLE_DEVICES": ""})
    if r.returncode == 3:
        pytest.skip("only without a GPU")
    assert r.returncode == 0 and r.stdout == "OK\n", r.stdout + r.stderr
