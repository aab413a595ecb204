"""Rows that gemm_stage_kernel straightens to the cache lines: no load outside the operand, every granule where it is looked for."""
import os
import subprocess

from paper_2003_06324_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_skewed_loads(tmp_path):
    exe = str(tmp_path / "skewed_load_bounds")
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-I" + build.INCLUDE, "-I" + build.CSRC,
                    "-x", "hip", os.path.join(HERE, "skewed_load_bounds.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, universal_newlines=True)
    assert r.returncode == 0, r.stdout
