"""Launch planning of the matrix-core pair kernel (csrc/pair_matrix.cpp) built
with g++ under AddressSanitizer and UndefinedBehaviorSanitizer: for some 400
windows and delay lists tests/host/mx_checks.cpp walks every read of every
task with the kernel's addresses, checks it against its plane, and compares the
sums with the plain definition, exactly. CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1209_3362_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_matrix_pair_planning(tmp_path):
    exe = str(tmp_path / "mx_checks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I" + CSRC,
                    os.path.join(ROOT, "tests", "host", "mx_checks.cpp"),
                    os.path.join(CSRC, "pair_matrix.cpp"), os.path.join(CSRC, "pair_plan.cpp"),
                    "-o", exe], check=True, capture_output=True, text=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert p.returncode == 0, p.stdout + p.stderr
    assert " 0 failures" in p.stdout
