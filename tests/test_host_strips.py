"""Builds (host only, no GPU) and runs the emulation of the strip kernels: reductions over dense blocks of narrow rows,
plain and fused, whose every element is folded once into the output where it belongs."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_strip_kernels_emulation(tmp_path):
    exe = tmp_path / "emulate_strips"
    csrc = os.path.join(ROOT, "paper_1810_08723_amd", "csrc")
    cmd = [HIPCC, "--cuda-host-only", "-O2", "-std=c++17", "-Wno-unused-command-line-argument", "-o", str(exe),
           os.path.join(ROOT, "tests", "host", "emulate_strips.hip"), os.path.join(csrc, "planner.cpp"),
           os.path.join(csrc, "red_launch.cpp")]
    subprocess.run(cmd, check=True, capture_output=True)
    r = subprocess.run([str(exe), "2500"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    assert r.stdout.startswith("ok:")
