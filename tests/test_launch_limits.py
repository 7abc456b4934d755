"""Launch limits of the kernels with more dynamic LDS than the default are state of a device:
every device that a handle is set up on gets them. Runs on the CPU, with the device objects of
the in-tree build and tests/launch_limits_driver.cpp."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2308_13476_amd", "csrc")
LIBDIR = os.path.join(ROOT, "paper_2308_13476_amd", "_lib")


def test_limits_are_raised_once_per_device(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    objs = [os.path.join(LIBDIR, o) for o in ("hm_level.o", "hm_setup.o", "hm_tail.o")]
    if not os.path.exists(hipcc) or not all(os.path.exists(o) for o in objs):
        pytest.skip("hipcc or the device objects are missing (run __graft_entry__.build())")
    drv, exe = tmp_path / "driver.o", tmp_path / "driver"
    subprocess.run([hipcc, "-x", "hip", "-c", os.path.join(ROOT, "tests", "launch_limits_driver.cpp"), "-o", str(drv),
                    "--offload-arch=gfx950", "-std=c++17", "-I", CSRC, "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops"], check=True, capture_output=True)
    subprocess.run([hipcc, str(drv)] + objs + ["-o", str(exe), "--offload-arch=gfx950"], check=True,
                   capture_output=True)
    res = subprocess.run([str(exe)], env=dict(os.environ, HIP_VISIBLE_DEVICES=""), capture_output=True, text=True,
                         timeout=120)
    assert res.returncode == 0, (res.returncode, res.stdout, res.stderr[-2000:])
