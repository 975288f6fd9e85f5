"""Host tables of the chunked k-point build (kpoint_tables.h), compiled by g++:
equal to one scan of the pair list per chunk, and made in one pass over it."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_tables_on_host(tmp_path):
    exe = str(tmp_path / "ktable_check")
    build = subprocess.run(["g++", "-std=c++17", "-O2", "-o", exe, os.path.join(HERE, "cpu_fft", "ktable_check.cpp")],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0, run.stdout[-4000:]
