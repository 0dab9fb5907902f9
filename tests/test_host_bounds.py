"""Device functions run on host threads with their buffers behind guard pages (tests/host):
every access of every thread of a workgroup stays inside its buffers."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")


def compile_host(source, out):
    """tests/host/<source> for the CPU, the kernel headers against the stand-in HIP header."""
    if not os.path.exists(CLANG):
        pytest.skip("needs the ROCm clang")
    subprocess.run([CLANG, "-x", "c++", "-std=c++20", "-O1", "-w", "-pthread", "-I" + HOST,
                    "-I" + os.path.join(ROOT, "paper_1602_08604_amd", "csrc"), os.path.join(HOST, source), "-o", str(out)],
                   check=True)
    return str(out)


@pytest.fixture(scope="module")
def tail_bounds(tmp_path_factory):
    return compile_host("tail_bounds.cpp", tmp_path_factory.mktemp("host") / "tail_bounds")


# F qubits left in the last pass: its own launch (a thread per column and (letters, outcomes)),
# and 3 qubits in the batch's tail stage of 256 threads.
@pytest.mark.parametrize("qubits,threads", [(1, 64), (2, 64), (3, 192), (4, 576), (3, 256)])
def test_last_pass_stays_in_bounds(tail_bounds, qubits, threads):
    run = subprocess.run([tail_bounds, str(qubits), str(threads)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr


def test_row_totals_stay_in_bounds(tmp_path):
    """The sub-tile pass with totals from the rows (6 to 8 qubits), its last row block."""
    run = subprocess.run([compile_host("subtile_rows.cpp", tmp_path / "subtile_rows")], capture_output=True, text=True,
                         timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
