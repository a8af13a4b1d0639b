"""The starts of the eigensolvers: fill_normal gives the values of std::normal_distribution bit for bit, so that starts of a
given seed stay what they were."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_14025_amd", "csrc")


def test_fill_normal_is_the_library_distribution(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path / "normal_driver"
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, os.path.join(HERE, "host", "normal_driver.cpp"),
                    os.path.join(CSRC, "hostla.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
