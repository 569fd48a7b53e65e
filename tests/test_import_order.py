"""One HIP runtime per process, whichever of torch and the package is imported first."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import {0}, {1}
print(len({{line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}}))
"""


@pytest.mark.parametrize("first,second", [("torch", "paper_2601_13631_amd"), ("paper_2601_13631_amd", "torch")])
def test_one_hip_runtime(first, second):
    r = subprocess.run([sys.executable, "-c", CODE.format(first, second)], cwd=ROOT, timeout=300,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == ["1"], r.stdout
