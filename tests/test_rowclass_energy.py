"""Pair energies of the grids whose FP64 planes are taken as classes of rows: the
z pass on the host (rowclass_energy_check, two and four classes, a ragged last
tile), and energies-only calls on the GPU with an odd number of pairs against the
oracle.  Tolerance: sums of 1e6 positive terms of three transforms, 1e-13 on the
host and 1e-12 of the largest energy on the GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_energy_body_on_host(tmp_path):
    exe = str(tmp_path / "rowclass_energy_check")
    build = subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(HERE, "cpu_fft"), "-o", exe,
                            os.path.join(HERE, "cpu_fft", "rowclass_energy_check.cpp")], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0, run.stdout[-4000:]


@pytest.mark.gpu
@pytest.mark.parametrize("n,npairs", [(100, 1), (100, 5), (108, 3), (120, 5)])
def test_pair_energies(lib, n, npairs):
    import torch

    import oracle
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] pair energies N={n}, {npairs} pairs", flush=True)
    L = 0.3 * n
    rng = np.random.default_rng(n)
    r = np.arange(n) * L / n
    phi = np.empty((4, n, n, n))
    for o in range(4):
        d = [(r - c * L + L / 2) % L - L / 2 for c in rng.random(3)]
        phi[o] = (np.exp(-0.5 * (d[0][:, None, None] ** 2 + d[1][None, :, None] ** 2 + d[2][None, None, :] ** 2) / 9.0)
                  + 0.01 * rng.standard_normal((n, n, n)))
    pairs = np.array([(0, 0), (0, 1), (1, 3), (2, 2), (2, 3)], dtype=np.int32)[:npairs]
    e = lib.Context().pair_energies(torch.as_tensor(phi, device="cuda"), torch.as_tensor(pairs, device="cuda"),
                                    Grid.cubic(n, L), kernel="erfc", omega=0.2, precision="fp64").cpu().numpy()
    ref = oracle.exchange_energy_pairs(phi, pairs, oracle.coulomb_kernel(n, L, "erfc", 0.2), (L / n) ** 3)
    np.testing.assert_allclose(e, ref, rtol=0, atol=1e-12 * np.abs(ref).max())
