"""The rules that choose a launch's shape, checked on the CPU at the points where both sides were measured."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_launch_rules(tmp_path):
    exe = tmp_path / "host_launch_rules"
    src = os.path.join(ROOT, "tests", "host_launch_rules.hip")
    build = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", src, "-o", str(exe)],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
    assert run.stdout.strip().endswith("ALL OK")
