"""The -inf fill of a group of logits (csrc/fill.h), compiled for the host."""

import shutil
import subprocess
from pathlib import Path

import pytest


def test_fill_group_on_the_host(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "fill"
    subprocess.run(["g++", "-O2", "-std=c++17", str(Path(__file__).parent / "fill" / "fill_driver.cpp"), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout)
