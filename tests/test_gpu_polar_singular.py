"""Columns that have no polar factor: A_C all zero, or with a NaN or an infinity in
it.  Both forms of the iteration (one workgroup up to 64 orbitals, tiles beyond)
must report it as not finite instead of taking it for converged."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bad", ["zero", "nan", "inf"])
@pytest.mark.parametrize("norb", [1, 17, 64, 65, 130])
def test_not_finite(lib, norb, bad):
    from paper_2101_03155_amd import AceError, Grid
    print(f"[gpu-case] singular columns norb={norb} {bad}", flush=True)
    n = 12
    g = torch.Generator(device="cuda").manual_seed(norb)
    psi = torch.randn(norb, n ** 3, dtype=torch.float64, device="cuda", generator=g)
    piv = torch.randperm(n ** 3, device="cuda", generator=g)[:norb]
    if bad == "zero":
        psi[:, piv] = 0.0
    else:
        psi[norb // 2, piv[norb // 3]] = float(bad)
    ctx, grid = lib.Context(), Grid.cubic(n, 5.0)
    with pytest.raises(AceError) as ei:
        ctx.localize_pivots(psi.reshape(norb, n, n, n), piv.to(torch.int32), grid)
    assert ei.value.status == "ACE_E_NONFINITE"
    # the context goes on working
    psi = torch.randn(norb, n ** 3, dtype=torch.float64, device="cuda", generator=g)
    psi[:, piv] = torch.eye(norb, dtype=torch.float64, device="cuda")
    U = ctx.localize_pivots(psi.reshape(norb, n, n, n), piv.to(torch.int32), grid)[1]
    assert float((U - torch.eye(norb, dtype=torch.float64, device="cuda")).abs().max()) <= 1e-12
