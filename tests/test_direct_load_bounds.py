"""No direct load of the tile kernels reads past its operand (but for the rest of the last dword), over K-slices,
remainders of K, straddled edges and leading dimensions below a granule: the addresses are walked on the CPU."""
import os
import subprocess

from paper_2003_06324_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_load_stays_inside_its_operand(tmp_path):
    exe = str(tmp_path / "direct_load_bounds")
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-I" + build.INCLUDE, "-I" + build.CSRC,
                    "-x", "hip", os.path.join(HERE, "direct_load_bounds.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, universal_newlines=True)
    assert r.returncode == 0, r.stdout
