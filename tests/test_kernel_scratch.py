"""No selection kernel keeps registers in scratch memory: their scores are held in
registers in earnest, up to 32 per thread."""
import os
import re
import subprocess

import pytest

from paper_2601_13631_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc here")
def test_selection_kernels_use_no_scratch(tmp_path):
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only",
                        "-c", os.path.join(build.CSRC, "select.hip"), "-o", str(tmp_path / "select.o")],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert len(names) == len(scratch) and sum("select" in x for x in names) >= 7
    assert not any(scratch), [x for x in zip(names, scratch) if x[1]]
