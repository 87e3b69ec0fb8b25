"""The lane set-up of the register-plane apply over all small mesh widths, and
the rule that chooses it, on the CPU: the header that the library uses,
compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_every_width_and_the_rule(tmp_path):
    exe = str(tmp_path / "lanes")
    subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
                    "-I" + os.path.join(ROOT, "paper_1911_01492_amd", "csrc"),
                    os.path.join(ROOT, "tests", "plane_lanes_driver.cpp"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "plane lanes: ok" in r.stdout
