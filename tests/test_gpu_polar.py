"""The Loewdin rotation on given columns at the edges of its two forms (one
workgroup up to 64 orbitals, 16 x 16 tiles beyond) against the polar factor
from an FP64 SVD, and the tile kernel at the edges of its quarters of K.

Tolerances: a polar factor moves by 2 eps |A| / (s_n + s_n-1) per rounding of A
and the products of the iteration sum up to 257 terms; singular values lie in
[0.3, 3] by construction, so 257 * 2.2e-16 * 3 / 0.3 = 6e-13 bounds it, and
1e-12 is asked.  Products: 300 roundings of the largest element, 1e-13."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("norb", [1, 2, 8, 15, 16, 17, 31, 48, 63, 64, 65, 80, 129, 257])
def test_rotation(lib, norb):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] polar norb={norb}", flush=True)
    n = 12
    g = torch.Generator(device="cuda").manual_seed(norb)
    rnd = lambda *s: torch.randn(*s, dtype=torch.float64, device="cuda", generator=g)  # noqa: E731
    q1, q2 = torch.linalg.qr(rnd(norb, norb))[0], torch.linalg.qr(rnd(norb, norb))[0]
    s = 0.3 + 2.7 * torch.rand(norb, dtype=torch.float64, device="cuda", generator=g)
    a = (q1 * s) @ q2.T
    piv = torch.randperm(n ** 3, device="cuda", generator=g)[:norb]
    psi = rnd(norb, n ** 3)
    psi[:, piv] = a
    phi, U = lib.Context().localize_pivots(psi.reshape(norb, n, n, n), piv.to(torch.int32), Grid.cubic(n, 5.0))
    ref = q1 @ q2.T
    err = float((U - ref).abs().max())
    print(f"  U {err:.2e}", flush=True)
    assert err <= 1e-12
    want = ref.T @ psi
    assert float((phi.reshape(norb, -1) - want).abs().max()) <= 1e-12 * float(psi.norm(dim=0).max())


@pytest.mark.parametrize("K,M", [(1, 1), (3, 4), (4, 16), (5, 17), (16, 15), (17, 33), (60, 64), (63, 3), (64, 65),
                                 (65, 40), (130, 70), (300, 20)])
def test_tile(lib, K, M):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] small product K={K} M={M}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K * 1000 + M)
    xi = torch.randn(K, 8, 8, 8, dtype=torch.float64, device="cuda", generator=g)
    x = torch.randn(M, 8, 8, 8, dtype=torch.float64, device="cuda", generator=g)
    grid = Grid.cubic(8, 2.4)
    y, _ = lib.Context().apply_energy(xi, x, grid)
    a, b = xi.reshape(K, -1), x.reshape(M, -1)
    c = grid.dV * (a @ b.T)
    scale = float((c.abs().T @ a.abs()).max())
    assert float((y.reshape(M, -1) + c.T @ a).abs().max()) <= 1e-13 * scale
