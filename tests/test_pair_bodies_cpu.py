"""Host builds of the pair-stage bodies (compiled by g++ against the host
stand-in for the HIP runtime header, run with one thread) against separable
naive DFTs over a whole field:

* kpoint_check: the k-point bodies (kpoint_phases.h), forward in-plane pass, z
  pass with v(|G + d|), inverse with accumulation (plain and conjugated), at
  one- and two-pass radix plans;
* rowclass_check: the row classes of the real owner path (pair_phases.h), two
  and four classes, both plan orders, ragged last tiles;
* owner_check: the owner pass with its product in the last transform pass and
  from the finished plane, against transform and product one after the other.

Tolerances: 1e-13 in FP64 (about 100 roundings of 1e-16 in six transforms of at
most 108 points), 1e-5 in FP32 likewise.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
@pytest.mark.parametrize("name", ["kpoint_check", "rowclass_check", "owner_check"])
def test_bodies_on_host(tmp_path, name):
    exe = str(tmp_path / name)
    build = subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(HERE, "cpu_fft"), "-o", exe,
                            os.path.join(HERE, "cpu_fft", name + ".cpp")], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0, run.stdout[-4000:]
