"""Host build of the k-point pair-stage bodies (kpoint_phases.h compiled by g++
against the host stand-in for the HIP runtime header, one thread): forward
in-plane pass, z pass with v(|G + d|), inverse with accumulation (plain and
conjugated) over a whole field against separable naive DFTs, at one- and
two-pass radix plans, to 1e-13 (about 100 roundings of 1e-16 in six
transforms of at most 64 points)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_kpoint_bodies_on_host(tmp_path):
    exe = str(tmp_path / "kpoint_check")
    build = subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(HERE, "cpu_fft"), "-o", exe,
                            os.path.join(HERE, "cpu_fft", "kpoint_check.cpp")], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0, run.stdout[-4000:]
