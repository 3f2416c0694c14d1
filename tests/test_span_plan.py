"""The device's rule for ending a launch, and the run driver's planning, against the
host controller, on the CPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(ROOT, "paper_2007_06134_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _check(name, tmp_path):
    """Build tests/native/<name>.cpp with the host controller and run it."""
    exe = str(tmp_path / name)
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-ffp-contract=off", "-I",
                        os.path.join(ROOT, "include"), "-I", SRC, os.path.join(HERE, "native", name + ".cpp"),
                        os.path.join(SRC, "controller.cpp"), "-o", exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("all ok"), r.stdout[-2000:] + r.stderr[-2000:]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_span_plan_follows_the_host_controller(tmp_path):
    _check("span_plan_check", tmp_path)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_driver_follows_the_host_controller(tmp_path):
    """The driver's launches and merged rows over random schedules (driver_check.cpp)."""
    _check("driver_check", tmp_path)
