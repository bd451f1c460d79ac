"""Host-side checks of the rules that choose a hopping launch (tests/host/launch_rules.cpp): which launches the
eight-threads-per-point kernel takes, and that an explicit launch configuration gets the kernel it asks for.  The C++
file includes the library's own header, so the rules checked are the ones the launches use."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def test_launch_rules_on_the_host(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = tmp_path / "launch_rules"
    build = subprocess.run([HIPCC, "-O2", "-std=c++17", "--cuda-host-only", "-x", "hip",
                            "-I", os.path.join(ROOT, "include"),
                            "-I", os.path.join(ROOT, "paper_1405_0700_amd", "csrc"),
                            os.path.join(ROOT, "tests", "host", "launch_rules.cpp"), "-o", str(exe)],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and run.stdout.strip() == "ok", run.stdout
