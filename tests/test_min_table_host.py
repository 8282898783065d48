"""The LDS table of minima (MinTable, paper_2607_20211_amd/csrc/drsf_dev.h) as
a workgroup uses it, on host threads: the committed header is compiled with g++
against stand-ins for the device built-ins it names, and one wave clears its
part of the table only after the others could have added to it.  No minimum may
be lost.  No GPU is used."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "min_table_host")


def test_no_minimum_is_lost_to_a_late_clear(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    (tmp_path / "hip").mkdir()
    shutil.copy(os.path.join(HERE, "hip_runtime_stub.h"), tmp_path / "hip" / "hip_runtime.h")
    exe = tmp_path / "min_table"
    cmd = [gxx, "-std=c++17", "-O1", f"-I{tmp_path}", f"-I{os.path.join(ROOT, 'paper_2607_20211_amd', 'csrc')}",
           os.path.join(HERE, "driver.cpp"), "-lpthread", "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
