"""The kernels' constant 1D operators agree with the tables that setup builds, on
the CPU (the library's host code, linked with its other objects)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
BUILD = os.path.join(ROOT, "paper_1911_01492_amd", "_build")
OTHERS = ("dg_affine", "dg_mfma", "dg_ppd", "dg_trilinear", "dg_vec", "dg_geom")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.skipif(not all(os.path.exists(os.path.join(BUILD, f + ".o")) for f in OTHERS),
                    reason="library objects not built")
def test_constant_tables_agree(tmp_path):
    exe = str(tmp_path / "tables")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_1911_01492_amd", "csrc"),
                    "-x", "hip", os.path.join(ROOT, "tests", "tables_driver.cpp"), "-x", "none"] +
                   [os.path.join(BUILD, f + ".o") for f in OTHERS] + ["-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "tables: ok" in r.stdout
    print(r.stdout)
