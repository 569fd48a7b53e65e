"""No source is compiled without NaN or infinity semantics.

The attention kernel redoes a slice whose outputs left fp32, which it sees by an
infinity or NaN among them: under -fno-honor-nans or the like that test may be
folded away.
"""
import os

from paper_2601_13631_amd import build


def test_no_reduced_float_semantics(monkeypatch, tmp_path):
    lines = []

    class Done:
        returncode, stderr = 0, ""

    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **_: lines.append(cmd) or Done)
    for src in build.SOURCES:
        build._compile(src, str(tmp_path))
    assert [os.path.basename(x) for line in lines for x in line if x.endswith(".hip")] == build.SOURCES
    for line in lines:
        bad = [x for x in line if x in ("-Ofast", "-fno-honor-nans", "-fno-honor-infinities")
               or x.startswith(("-ffast-math", "-ffinite-math", "-menable-no"))]
        assert not bad, bad
