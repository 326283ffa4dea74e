"""The bf16-matrix Conv2d kernel's staging (unit columns, guards, clipping, plan)
on the CPU with whole numbers: every plan of a sweep of kernels, strides, pads
and widths gives the gradient of the definition, reads inside its planes and
adds every backprop to the bias once."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2109_12298_amd", "csrc")


def test_conv_staging_matches_definition(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "conv_staging")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-I", CSRC, "-o", exe, os.path.join(HERE, "conv_staging_ref.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-2000:]
