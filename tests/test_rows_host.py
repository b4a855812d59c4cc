"""Row programs (csrc/closed.cpp) with rows as long as a node recorded in many
columns would give the adjoint's gather: kept whole, or refused."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1903_01081_amd", "csrc")


def test_long_rows_are_kept_whole_or_refused(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path / "rows_driver")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(CSRC, "closed.cpp"), os.path.join(ROOT, "tests", "host_asan", "rows_driver.cpp"),
                        "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([out], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout == "ok\n", (r.stdout[-2000:], r.stderr[-3000:])
