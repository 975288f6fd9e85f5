"""Small grids: the candidate pool drawn by one workgroup (fewer columns than
the pool holds, a little more, many more; beyond 65536 columns the kernels of
large grids) against greedy pivoting by LAPACK, and the split products with
short chunks of K against torch in FP64.

Pivots are whole numbers and equal: random columns leave no ties.  Products:
1e-13 of the largest element for sums of at most 110592 positive terms in
chunks (random-walk rounding below 1e-15 each)."""
import numpy as np
import pytest
import scipy.linalg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("norb,n", [(1, 8), (5, 8), (16, 12), (20, 16), (40, 24), (70, 32), (30, 48)])
def test_pivots(lib, norb, n):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] pool norb={norb} N={n}", flush=True)
    rng = np.random.default_rng(norb * 100 + n)
    psi = rng.normal(size=(norb, n ** 3)) * np.exp(-3.0 * rng.random(n ** 3))
    _, _, want = scipy.linalg.qr(psi, mode="economic", pivoting=True)
    phi, piv, U = lib.Context().localize(torch.as_tensor(psi.reshape(norb, n, n, n), device="cuda"),
                                         Grid.cubic(n, 6.0))
    np.testing.assert_array_equal(piv.cpu().numpy(), want[:norb])


@pytest.mark.parametrize("norb,n", [(1, 8), (3, 12), (8, 24), (100, 24), (130, 32), (20, 48)])
def test_overlaps(lib, norb, n):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] overlaps norb={norb} N={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(norb + n)
    phi = torch.randn(norb, n, n, n, dtype=torch.float64, device="cuda", generator=g)
    grid = Grid.cubic(n, 6.0)
    pairs, o = lib.Context().pairlist(phi, grid, 0.0)
    a = phi.reshape(norb, -1).abs()
    want = grid.dV * (a @ a.T)
    iu = torch.triu_indices(norb, norb, device="cuda")
    assert torch.equal(pairs.long().T, iu)
    assert float((o - want[iu[0], iu[1]]).abs().max()) <= 1e-13 * float(want.max())
