"""The Gram sums of a GMRES(3) step (§5.3) are one row per block of the pass that forms the Krylov
vectors, in a region of fixed size. tests/partial_sums_driver.cpp computes the blocks of these
passes for every grid, cap, block height and batch size. Runs on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2308_13476_amd", "csrc")


def test_gram_sums_of_every_grid_fit_their_region(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    drv, exe = tmp_path / "driver.o", tmp_path / "driver"
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-c", os.path.join(ROOT, "tests", "partial_sums_driver.cpp"),
                    "-o", str(drv), "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC], check=True,
                   capture_output=True)
    subprocess.run([hipcc, str(drv), "-o", str(exe), "--offload-arch=gfx950"], check=True, capture_output=True)
    res = subprocess.run([str(exe)], env=dict(os.environ, HIP_VISIBLE_DEVICES=""), capture_output=True, text=True,
                         timeout=300)
    assert res.returncode == 0, res.stdout[-2000:]
