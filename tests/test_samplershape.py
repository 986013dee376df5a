"""Host check of the samplers' launch shape (csrc/samplershape.hpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_a_shape_that_is_set_is_taken_as_given(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "samplershape_check")
    subprocess.run([gxx, "-O1", "-std=c++17", os.path.join(HERE, "samplershape_check.cpp"), "-o", exe], check=True,
                   capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
