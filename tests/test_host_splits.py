"""Host-side check of the kernels' grid splits: compiles tests/splits_check.cpp against the
package header with g++ and runs it (plain integer arithmetic; no oracle is involved)."""
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_07915_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_grid_splits():
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "splits_check")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover", f"-I{CSRC}",
                        os.path.join(ROOT, "tests", "splits_check.cpp"), "-o", exe], check=True)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr
