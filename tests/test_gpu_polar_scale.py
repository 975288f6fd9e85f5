"""The Loewdin rotation does not depend on the scale of its columns: orbitals in
units that make them very small or large (squares still in range, cubes not) give
the rotation of the unscaled ones.  Scaling by a power of two changes no rounding of
the scaled iterate, so the bound is the rotation's own (1e-12 for singular values
in [0.3, 3] and up to 257 terms per sum)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("norb", [1, 64, 65, 200])
@pytest.mark.parametrize("power", [-400, -350, 350, 400])
def test_rotation(lib, norb, power):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] polar norb={norb} scale 2^{power}", flush=True)
    n = 12
    g = torch.Generator(device="cuda").manual_seed(norb)
    rnd = lambda *s: torch.randn(*s, dtype=torch.float64, device="cuda", generator=g)  # noqa: E731
    q1, q2 = torch.linalg.qr(rnd(norb, norb))[0], torch.linalg.qr(rnd(norb, norb))[0]
    a = (q1 * (0.3 + 2.7 * torch.rand(norb, dtype=torch.float64, device="cuda", generator=g))) @ q2.T
    piv = torch.randperm(n ** 3, device="cuda", generator=g)[:norb]
    psi = rnd(norb, n ** 3)
    psi[:, piv] = a
    psi = psi * 2.0 ** power
    U = lib.Context().localize_pivots(psi.reshape(norb, n, n, n), piv.to(torch.int32), Grid.cubic(n, 5.0))[1]
    assert float((U - q1 @ q2.T).abs().max()) <= 1e-12
