"""Host check of the row starts of the edge-list ingest (csrc/rowstarts.hpp),
compiled for the CPU with AddressSanitizer and UndefinedBehaviorSanitizer: no
pair kept, one, and the sizes around a block's 1024 entries."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rowstarts_exe(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("rowstarts") / "rowstarts_check")
    subprocess.run([gxx, "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(HERE, "rowstarts_check.cpp"),
                    "-o", exe], check=True, capture_output=True)
    return exe


@pytest.mark.parametrize("n", [1, 30, 5000])
@pytest.mark.parametrize("K", [0, 1, 2, 255, 1023, 1024, 1025, 4096])
def test_starts_count_the_keys_below(rowstarts_exe, K, n):
    r = subprocess.run([rowstarts_exe, str(K), str(n), str(K + n)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
