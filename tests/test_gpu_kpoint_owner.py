"""Owner-computes pair stage of the k-point build against its split passes and
in chunks: the grids where one route ends and the other begins, spectra budgets
that force one slot-chunk or many, and a workspace cap."""
import os

import numpy as np
import pytest

from oracle import kpoint_oracle as ko
from synth import SystemSpec, make_bloch_orbitals

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(n, nmol, kf):
    from paper_2101_03155_amd import Grid
    spec = SystemSpec(n_mol=nmol, L=0.45 * n, N=n, sigma=0.8, offset=0.7, placement="uniform", seed=600 + n)
    u, kv = make_bloch_orbitals(spec, kf)
    return spec, Grid.cubic(n, spec.L), u, [tuple(k) for k in kv], ko.full_pairs(len(u)).astype(np.int32)


def _run(lib, monkeypatch, case, budget=None, cap=None):
    spec, grid, u, kv, pairs = case
    for key, v in (("ACE_OWNER_SPECTRA_MAX", budget), ("ACE_WORKSPACE_MAX", cap)):
        monkeypatch.delenv(key, raising=False)
        if v is not None:
            monkeypatch.setenv(key, str(v))
    ctx = lib.Context()
    r = ctx.build_kpoints(torch.as_tensor(u, device="cuda"), kv, spec.norb, torch.as_tensor(pairs, device="cuda"),
                          grid, kernel="erfc", omega=0.5, want_W=True)
    out = {k: r[k].cpu().numpy() for k in ("W", "M", "xi", "ex")}
    ctx.close()
    return out


def _same(a, b, tol, what):
    for k in a:
        err = np.abs(a[k] - b[k]).max() / np.abs(b[k]).max()
        print(f"  {what} {k}: {err:.2e}", flush=True)
        assert err <= tol, (what, k)


# tolerances: W and M to 1e-12 of their largest element, as the parity suite; xi to 1e-10
@pytest.mark.parametrize("n,nmol,kf", [(8, 1, [(0, 0, 0), (0.5, 0, 0)]), (80, 1, [(0, 0, 0), (0, 0.5, 0)]),
                                       (96, 1, [(0, 0, 0)]), (100, 1, [(0, 0, 0)])])
def test_grids_against_the_oracle(lib, monkeypatch, n, nmol, kf):
    print(f"[gpu-case] k-point owner route N={n}", flush=True)
    case = _case(n, nmol, kf)
    spec, _, u, kv, pairs = case
    got = _run(lib, monkeypatch, case)
    ref = ko.ace_build_k(u, np.array(kv), spec.norb, pairs, n, spec.L, "erfc", 0.5)
    for k, tol in (("W", 1e-12), ("M", 1e-12), ("xi", 1e-10)):
        err = np.abs(got[k] - ref[k]).max() / np.abs(ref[k]).max()
        print(f"  {k}: {err:.2e}", flush=True)
        assert err <= tol, k
    assert abs(got["ex"][0] - ref["ex"]) <= 1e-10 * abs(ref["ex"])


def test_chunked_spectra_and_workspace_cap(lib, monkeypatch):
    print("[gpu-case] k-point owner route, chunked spectra", flush=True)
    n = 24
    case = _case(n, 3, [(0, 0, 0), (0.5, 0, 0), (0, 0.5, 0)])  # 36 orbitals, 666 pairs
    slot = n ** 3 * 16
    whole = _run(lib, monkeypatch, case)
    for budget in (0, 100 * slot + 1, 665 * slot):  # 32 slots at a time; 100; all but one
        _same(_run(lib, monkeypatch, case, budget=budget), whole, 1e-12, f"budget {budget}")
    # a workspace cap below what all spectra take, and the same build still runs
    _same(_run(lib, monkeypatch, case, cap=60 << 20), whole, 1e-12, "workspace cap")
