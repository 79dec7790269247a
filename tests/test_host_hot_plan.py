"""Host logic without a GPU: the choice of the hot-column layout's row blocks,
built from the library's own header with g++, plain and under sanitizers."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2001_07938_amd", "csrc")


@pytest.mark.parametrize("san", [[], ["-fsanitize=address,undefined"]], ids=["plain", "asan"])
def test_hot_blocks(tmp_path, san):
    exe = tmp_path / "hot_plan_test"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wextra", *san, f"-I{CSRC}",
                           os.path.join(ROOT, "tests", "host", "hot_plan_test.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, UBSAN_OPTIONS="halt_on_error=1"))
    assert r.returncode == 0, r.stdout + r.stderr
    assert "hot plan ok" in r.stdout
