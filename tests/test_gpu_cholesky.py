"""Cholesky factor and inverse at the edges of their blocks (16-column panels,
the one-workgroup limit of 128, ragged 128-column blocks up to 512).

The factor alone: the condition number that localize_step reports, from the
diagonal of the factor of A_C^T A_C, against QR in FP64.  With |A| = 3, singular
values in [0.3, 3] the Gram matrix has condition 100; its factor's diagonal is
exact to 512 * 2.2e-16 * 100 = 1e-11 relative, 1e-9 is asked of the ratio squared.
The inverse: xi = L^-1 W of a build over all pairs, dV xi phi^T = +-L^T (tolerance
and reason as for the triangular product's test)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("norb", [1, 2, 15, 16, 17, 64, 65, 127, 128, 129, 144, 256, 257, 300, 511])
def test_factor(lib, norb):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] factor norb={norb}", flush=True)
    n = 12
    g = torch.Generator(device="cuda").manual_seed(norb)
    rnd = lambda *s: torch.randn(*s, dtype=torch.float64, device="cuda", generator=g)  # noqa: E731
    q1, q2 = torch.linalg.qr(rnd(norb, norb))[0], torch.linalg.qr(rnd(norb, norb))[0]
    a = (q1 * (0.3 + 2.7 * torch.rand(norb, dtype=torch.float64, device="cuda", generator=g))) @ q2.T
    piv = torch.randperm(n ** 3, device="cuda", generator=g)[:norb]
    psi = 0.1 * rnd(norb, n ** 3)
    psi[:, piv] = a
    info = lib.Context().localize_step(psi.reshape(norb, n, n, n), piv.to(torch.int32), Grid.cubic(n, 5.0), 1e300)[3]
    d = torch.linalg.qr(a.cpu())[1].diagonal().abs()
    want = float((d.max() / d.min()) ** 2)
    assert info["reused_columns"]
    assert abs(info["gram_cond"] - want) <= 1e-9 * want


@pytest.mark.parametrize("norb,n", [(1, 8), (2, 8), (15, 8), (33, 8), (112, 12), (128, 12), (130, 12), (300, 12),
                                    (385, 12)])
def test_inverse(lib, norb, n):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] inverse norb={norb}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(norb)
    phi = torch.randn(norb, n, n, n, dtype=torch.float64, device="cuda", generator=g)
    pairs = torch.triu_indices(norb, norb, device="cuda").T.to(torch.int32).contiguous()
    grid = Grid.cubic(n, 9.0)
    r = lib.Context().build(phi, pairs, grid, kernel="erfc", omega=0.3, precision="fp64")
    t = grid.dV * (r["xi"].reshape(norb, -1) @ phi.reshape(norb, -1).T)
    m = t.T @ t
    scale = float(r["M"].abs().max())
    low = float(torch.tril(t, -1).abs().max()) / float(t.abs().max())
    err = min(float((m + r["M"]).abs().max()), float((m - r["M"]).abs().max())) / scale
    print(f"  lower {low:.2e} product {err:.2e}", flush=True)
    assert low <= 1e-10 and err <= 1e-10
