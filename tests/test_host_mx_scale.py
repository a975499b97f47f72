"""Scale of the matrix-core pair kernel's whole numbers (tests/host/mx_scale_checks.cpp),
built with g++ under AddressSanitizer and UndefinedBehaviorSanitizer. CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1209_3362_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_whole_numbers_and_sums_fit(tmp_path):
    exe = str(tmp_path / "mx_scale_checks")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I" + CSRC, "-I" + os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "host", "mx_scale_checks.cpp"),
                    *(os.path.join(CSRC, f) for f in
                      ("pair_matrix.cpp", "pair_plan.cpp")), "-o", exe],
                   check=True, capture_output=True, text=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert p.returncode == 0, p.stdout + p.stderr
    assert " 0 failures" in p.stdout
