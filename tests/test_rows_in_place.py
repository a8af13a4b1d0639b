"""Which rows of a caller the kernels use in place: only memory of the system's own device (rows on another GPU go through
a copy, as a kernel may not be able to reach them). The rule is host code, checked over memory kinds, devices and
addresses; that rows_in and rows_out ask it, and ask the runtime where the memory is, in the source."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_14025_amd", "csrc")


def test_rule(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path / "rows_driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, os.path.join(HERE, "host", "rows_driver.cpp"),
                    "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_rows_ask_the_rule():
    src = open(os.path.join(CSRC, "system.cpp")).read()
    body = {f: re.search(r"static [a-z]+ " + f + r"\(.*?\n}\n", src, re.S).group(0) for f in ("direct_rows", "rows_in", "rows_out")}
    assert "hipPointerGetAttributes" in body["direct_rows"] and "rows_in_place(" in body["direct_rows"]
    for f in ("rows_in", "rows_out"):
        assert "direct_rows(S, " in body[f]
