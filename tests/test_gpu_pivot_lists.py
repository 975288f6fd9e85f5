"""Pivot search whose pools alternate between refreshing a list of columns and all
of them: strong columns among weak ones, a slab in vacuum, steps of the column
norms, each with residuals that fall at several rates.  The pivots must be greedy
QRCP's, step by step: with the earlier pivot columns projected out, no column's
residual norm exceeds the picked one's by more than rounding (1e-10 of the
largest initial norm)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _orbitals(kind, norb, n, g):
    ng = n ** 3
    x = torch.randn(norb, ng, dtype=torch.float64, device="cuda", generator=g)
    u = torch.rand(ng, dtype=torch.float64, device="cuda", generator=g)
    if kind == "peaks":
        w = torch.where(u < 0.5 * norb / ng, 3.0, 0.05)
    elif kind == "slab":
        z = torch.arange(n, device="cuda", dtype=torch.float64).repeat_interleave(n * n) / n
        w = torch.exp(-((z - 0.5) / 0.1) ** 2)
    else:  # steps: a tenth of the columns at 1, a fifth at 1/4, the rest at 1/16
        w = torch.where(u < 0.1, 1.0, torch.where(u < 0.3, 0.25, 0.0625))
    q, _ = torch.linalg.qr((x * w).T)
    return q.T.contiguous().reshape(norb, n, n, n)


@pytest.mark.parametrize("kind", ["peaks", "slab", "steps"])
@pytest.mark.parametrize("norb,n", [(60, 32), (256, 32), (200, 48), (400, 32)])
def test_pivots_are_greedy(lib, kind, norb, n):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] pivots {kind} norb={norb} N={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(norb)
    psi = _orbitals(kind, norb, n, g)
    phi, piv, U = lib.Context().localize(psi, Grid.cubic(n, 0.3 * n))
    R = psi.reshape(norb, -1).clone()
    scale = float((R * R).sum(0).max())
    assert len(set(piv.tolist())) == norb
    for k, p in enumerate(piv.tolist()):
        r2 = (R * R).sum(0)
        assert float(r2.max()) <= float(r2[p]) + 1e-10 * scale, (k, float(r2[p]), float(r2.max()))
        q = R[:, p] / R[:, p].norm()
        R -= torch.outer(q, q @ R)
        R -= torch.outer(q, q @ R)
    assert float((U.T @ U - torch.eye(norb, dtype=torch.float64, device="cuda")).abs().max()) < 1e-12
