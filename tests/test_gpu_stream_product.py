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
