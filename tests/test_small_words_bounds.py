"""Rows that gemm_small_kernel reads word by word: no read outside the operand, every element in its place."""
import os
import subprocess

from paper_2003_06324_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_word_reads(tmp_path):
    exe = str(tmp_path / "small_words_bounds")
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-I" + build.INCLUDE, "-I" + build.CSRC,
                    "-x", "hip", os.path.join(HERE, "small_words_bounds.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, universal_newlines=True)
    assert r.returncode == 0, r.stdout
