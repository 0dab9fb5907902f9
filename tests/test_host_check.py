"""The built library with the HIP runtime's calls replaced by a program's own (tests/host):
what its entry points do when the host's copies or its memory fail."""
import os
import subprocess

import pytest

from paper_1602_08604_amd import lre as L
from tests.test_host_bounds import CLANG, HOST, ROOT

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm clang")


def run_host(source, tmp_path):
    exe = str(tmp_path / "host")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-rdynamic", "-I" + os.path.join(ROOT, "include"),
                    os.path.join(HOST, source), "-o", exe, "-ldl"], check=True)
    run = subprocess.run([exe, L.LIB_PATH], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr


def test_an_error_survives_a_failed_copy(tmp_path):
    run_host("check_flags.cpp", tmp_path)


def test_no_exception_when_host_memory_runs_out(tmp_path):
    run_host("no_memory.cpp", tmp_path)
