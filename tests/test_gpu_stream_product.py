"""The streaming left-small product (C = S B with S in registers) at the edges
of its shapes, through the application of the operator (y = -(dV xi x^T)^T xi, K =
projectors, M = functions): one row, the 16-row blocks, the 64- and 128-row
workgroups, several of them, K at the limits of each variant, column counts that
leave a ragged last tile, against FP64 torch.  Tolerance: sums of at most 256
products, 1e-13 of the largest element (256 roundings of 1e-16 at most)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("K,M", [(1, 1), (3, 17), (16, 64), (64, 64), (64, 65), (65, 16), (100, 33), (128, 128),
                                 (128, 130), (127, 257), (40, 300), (193, 193), (256, 256), (255, 200), (192, 192)])
@pytest.mark.parametrize("n", [12, 24])
def test_shapes(lib, K, M, n):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] streaming product K={K} M={M} N={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K * 1000 + M)
    xi = torch.randn(K, n, n, n, dtype=torch.float64, device="cuda", generator=g)
    x = torch.randn(M, n, n, n, dtype=torch.float64, device="cuda", generator=g)
    grid = Grid.cubic(n, 0.3 * n)
    y, _ = lib.Context().apply_energy(xi, x, grid)
    a, b = xi.reshape(K, -1), x.reshape(M, -1)
    c = grid.dV * (a @ b.T)
    ref = -(c.T @ a)
    # the error of c (1e-15 relative to its terms) is not this product's: compare with the product's own scale
    scale = float((c.abs().T @ a.abs()).max())
    err = float((y.reshape(M, -1) - ref).abs().max())
    print(f"  err {err / scale:.2e}", flush=True)
    assert err <= 1e-13 * scale


@pytest.mark.parametrize("norb", [17, 64, 65, 127, 129, 161, 192, 193, 208, 225, 256, 257])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_triangular(lib, norb, precision):
    """xi = L^-1 W of a build, L from M = dV phi W^T: the rows below and above 128
    run as two launches.  Checked without L, with all pairs (M is then symmetric):
    xi phi^T dV = +-L^T, so that its lower part vanishes and L L^T = |M|.  W has
    the rounding of the build's precision, so that M is symmetric to about 1e-15
    or 1e-7 of its largest element; 1e-10 and 2e-6 leave room for the condition of
    M (below 1e3 for random orbitals) in FP64 and for a few roundings in FP32."""
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] triangular product norb={norb} {precision}", flush=True)
    n, L = 16, 9.0
    g = torch.Generator(device="cuda").manual_seed(norb)
    phi = torch.randn(norb, n, n, n, dtype=torch.float64, device="cuda", generator=g)
    pairs = torch.triu_indices(norb, norb, device="cuda").T.to(torch.int32).contiguous()
    grid = Grid.cubic(n, L)
    r = lib.Context().build(phi, pairs, grid, kernel="erfc", omega=0.3, precision=precision)
    t = grid.dV * (r["xi"].reshape(norb, -1) @ phi.reshape(norb, -1).T)
    m = t.T @ t
    scale = float(r["M"].abs().max())
    low = float(torch.tril(t, -1).abs().max()) / float(t.abs().max())
    tol = 1e-10 if precision == "fp64" else 2e-6
    err = min(float((m + r["M"]).abs().max()), float((m - r["M"]).abs().max())) / scale
    print(f"  lower {low:.2e} product {err:.2e}", flush=True)
    assert low <= tol and err <= tol
