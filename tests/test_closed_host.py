"""The closed-form plan of the one-workgroup solve (csrc/closed.cpp) on the
CPU, under AddressSanitizer and UndefinedBehaviorSanitizer: sizes, index
ranges and the solution its row programs give against a dense solve, for
every kind of cut (none, some, the whole component) and workgroup size."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1903_01081_amd", "csrc")


def test_closed_plan_solves_under_sanitizers(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path / "closed_driver")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "analysis.cpp"),
                        os.path.join(CSRC, "closed.cpp"), os.path.join(ROOT, "tests", "host_asan", "closed_driver.cpp"),
                        "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([out], capture_output=True, text=True, timeout=600, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), (r.stdout[-2000:], r.stderr[-3000:])
