"""The address rules of the slim form of the dense products, walked on the CPU: every load inside its operand or cut off,
every operand of a matrix instruction the element the definition of the product puts there; planted mistakes are noticed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_02885_amd", "csrc")
# bf16, dx, tile, R, Q, Kd
CASES = [(b, dx, t, *s) for b, dx, t in ((0, 0, 32), (0, 1, 32), (1, 0, 32), (1, 1, 32), (1, 0, 64))
         for s in ((1, 1, 1), (31, 33, 63), (32, 32, 64), (33, 31, 65), (70, 100, 1030), (128, 65, 520))]


def test_the_walk_passes_and_notices_planted_mistakes(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc to compile the driver with")

    def run(plant):
        exe = str(tmp_path / f"slim{plant}")
        subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", f"-DPACK_HALO_PLANT={plant}", "-I", CSRC,
                        os.path.join(CSRC, "gemm_fetch_check.cpp"), os.path.join(ROOT, "tests", "slim_walk_driver.cpp"), "-o", exe],
                       check=True, capture_output=True)
        return [subprocess.run([exe, *map(str, c)], capture_output=True, text=True) for c in CASES]

    for c, r in zip(CASES, run(0)):
        assert r.returncode == 0 and r.stdout.startswith("OK"), (c, r.stdout)
    for plant in (11, 12):   # a row loaded from its neighbour, the two halves of a transposing read swapped
        assert any(r.returncode == 1 and "FAIL" in r.stdout for r in run(plant)), plant
