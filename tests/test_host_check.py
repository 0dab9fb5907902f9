"""lre_check where the host's copies fail: the built library with the HIP runtime's calls
replaced by a program's own (tests/host/check_flags.cpp)."""
import os
import subprocess

from paper_1602_08604_amd import lre as L
from tests.test_host_bounds import CLANG, HOST, ROOT

import pytest


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm clang")
def test_an_error_survives_a_failed_copy(tmp_path):
    exe = str(tmp_path / "check_flags")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-rdynamic", "-I" + os.path.join(ROOT, "include"),
                    os.path.join(HOST, "check_flags.cpp"), "-o", exe, "-ldl"], check=True)
    run = subprocess.run([exe, L.LIB_PATH], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
