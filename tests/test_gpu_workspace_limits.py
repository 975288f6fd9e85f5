"""Calls under ACE_WORKSPACE_MAX, and what a context holds between calls: a path that
keeps the spectra of all pairs gives way to one that fits, spectra of an earlier
call give way to what this one needs, and the real and the k-point build keep
their spectra in one place."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MB = 1 << 20


def _ctx(lib, monkeypatch, cap):
    monkeypatch.setenv("ACE_WORKSPACE_MAX", str(cap))
    ctx = lib.Context()
    monkeypatch.delenv("ACE_WORKSPACE_MAX")
    return ctx


def _orbitals(norb, n, seed, cplx=False):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(norb, n, n, n, dtype=torch.complex128 if cplx else torch.float64, device="cuda", generator=g)


def _full(n):
    return torch.triu_indices(n, n, device="cuda").T.to(torch.int32).contiguous()


# spectra of all pairs / what the passes of one launch need beside them, MB: 160^3
# 36 x 33 / 262 + 262 for W; 96^3 78 x 7 / 85 + 85; 48^3 in FP32 136 x 0.45 / 22
@pytest.mark.parametrize("norb,n,prec,cap", [(8, 160, "fp64", 700), (12, 96, "fp64", 300), (16, 48, "fp32", 56)])
def test_build_gives_way_to_the_rounds(lib, monkeypatch, norb, n, prec, cap):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] capped build norb={norb} N={n} {prec}", flush=True)
    phi, pairs, grid = _orbitals(norb, n, norb), _full(norb), Grid.cubic(n, 0.2 * n)
    ref = lib.Context().build(phi, pairs, grid, kernel="erfc", omega=0.3, precision=prec, want_W=True)
    ctx = _ctx(lib, monkeypatch, cap * MB)
    tol = 1e-12 if prec == "fp64" else 1e-5
    for _ in range(2):
        r = ctx.build(phi, pairs, grid, kernel="erfc", omega=0.3, precision=prec, want_W=True)
        for k in ("W", "M"):
            assert float((r[k] - ref[k]).abs().max()) <= tol * float(ref[k].abs().max()), k
    # where all fits again the resident form runs: a tenth of the pairs
    few = pairs[:: 10].contiguous()
    a = ctx.pair_energies(phi, few, grid, kernel="erfc", omega=0.3, precision=prec)
    b = lib.Context().pair_energies(phi, few, grid, kernel="erfc", omega=0.3, precision=prec)
    assert float((a - b).abs().max()) <= tol * float(b.abs().max())


def test_spectra_in_one_place(lib):
    from paper_2101_03155_amd import Grid
    print("[gpu-case] spectra held between calls", flush=True)
    ctx, g = lib.Context(), Grid.cubic(48, 20.0)
    u, phi, pairs = _orbitals(24, 48, 1, True), _orbitals(24, 48, 2), _full(24)
    ctx.build(phi[:2], _full(2), g, kernel="erfc", omega=0.3)
    ctx.build_kpoints(u, [(0.0, 0.0, 0.0)], 24, pairs, g, kernel="erfc", omega=0.3)  # 300 spectra, 531 MB
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    r = ctx.build(phi, pairs, g, kernel="erfc", omega=0.3)  # 300 half spectra, 276 MB; W 21 MB
    torch.cuda.synchronize()
    more = before - torch.cuda.mem_get_info()[0]
    print(f"  {more / MB:.0f} MB more", flush=True)
    assert more <= 128 * MB
    del r


def test_held_spectra_give_way(lib, monkeypatch):
    from paper_2101_03155_amd import Grid
    print("[gpu-case] capped context, spectra of an earlier call", flush=True)
    # 8 Bloch orbitals on 48^3: 36 spectra of 1.8 MB = 64 MB, fields 35 MB; then 512
    # on 12^3, whose tables and partial sums need some 20 MB more, and a real build
    ctx = _ctx(lib, monkeypatch, 104 * MB)
    u = _orbitals(8, 48, 1, True)
    kv = [(0.0, 0.0, 0.0), (0.5, 0.0, 0.0), (0.0, 0.5, 0.0), (0.0, 0.0, 0.5)]
    ctx.build_kpoints(u, kv[:2], 4, _full(8), Grid.cubic(48, 20.0), kernel="erfc", omega=0.3)
    u, pairs = _orbitals(512, 12, 2, True), _full(512)
    g = Grid.cubic(12, 6.0)
    r = ctx.build_kpoints(u, kv, 128, pairs, g, kernel="erfc", omega=0.3, want_W=True)
    ref = lib.Context().build_kpoints(u, kv, 128, pairs, g, kernel="erfc", omega=0.3, want_W=True)
    for k in ("W", "M"):
        assert float((r[k] - ref[k]).abs().max()) <= 1e-12 * float(ref[k].abs().max()), k
    # 10 on 48^3: beside the tables held by now 32 spectra no longer fit
    u, g = _orbitals(10, 48, 4, True), Grid.cubic(48, 20.0)
    r = ctx.build_kpoints(u, kv[:2], 5, _full(10), g, kernel="erfc", omega=0.3, want_W=True)
    ref = lib.Context().build_kpoints(u, kv[:2], 5, _full(10), g, kernel="erfc", omega=0.3, want_W=True)
    assert float((r["W"] - ref["W"]).abs().max()) <= 1e-12 * float(ref["W"].abs().max())
    phi, few = _orbitals(40, 32, 3), _full(40)
    g = Grid.cubic(32, 9.0)
    r = ctx.build(phi, few, g, kernel="erfc", omega=0.3, want_W=True)
    ref = lib.Context().build(phi, few, g, kernel="erfc", omega=0.3, want_W=True)
    assert float((r["W"] - ref["W"]).abs().max()) <= 1e-12 * float(ref["W"].abs().max())


def test_partial_sums_give_way(lib, monkeypatch):
    from paper_2101_03155_amd import Grid
    print("[gpu-case] capped products on a small grid", flush=True)
    # 256 orbitals on 24^3: 54 partial products of 0.5 MB fit in the cap, 108 do not
    phi, g = _orbitals(256, 24, 5), Grid.cubic(24, 9.0)
    ctx = _ctx(lib, monkeypatch, 40 * MB)
    pairs, o = ctx.pairlist(phi, g, 0.0)
    want_p, want_o = lib.Context().pairlist(phi, g, 0.0)
    assert torch.equal(pairs, want_p)
    assert float((o - want_o).abs().max()) <= 1e-13 * float(want_o.abs().max())
    y, ex = _ctx(lib, monkeypatch, 40 * MB).apply_energy(phi, phi, g)
    want_y, want_ex = lib.Context().apply_energy(phi, phi, g)
    assert float((y - want_y).abs().max()) <= 1e-12 * float(want_y.abs().max())
    assert np.isclose(float(ex), float(want_ex), rtol=1e-12)
