"""Selection by threshold and the ordered pair lists at the edges of their
workgroups (below one wave, around 1024 pairs, several elements per thread),
against a sort on the host, and the orbital moments with fused subsampling at
the grid sizes where lanes own one, two, three or four columns.

Lists are whole numbers and must be equal: budgets and cut-offs are put midway
between two neighbouring partial sums or values, far from any rounding.
Feature tolerances are those of single precision (2^-24 relative on lengths,
times a few operations; logarithms of sums rounded once to single precision)."""
import numpy as np
import pytest

from oracle import screener_oracle as so

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _orbitals(norb, n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(norb, n, n, n, dtype=torch.float64, device="cuda", generator=g)


@pytest.mark.parametrize("norb", [1, 2, 11, 44, 45, 91, 256, 300])
def test_lists(lib, norb):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] selection norb={norb}", flush=True)
    ctx, g = lib.Context(), Grid.cubic(8, 6.0)
    phi = _orbitals(norb, 8, norb)
    iu, ju = np.triu_indices(norb)
    every = np.stack([iu, ju], 1)
    off = iu != ju
    # overlap rule
    a = phi.reshape(norb, -1).abs()
    O = (g.dV * (a @ a.T)).cpu().numpy()[iu, ju]
    s = np.sort(O[off])
    cuts = [1e9]
    if off.any():
        mid = 0.5 * (s[1:] + s[:-1])
        cuts += [0.5 * s[0]] + [mid[int(f * (len(mid) - 1))] for f in (0.0, 0.3, 1.0) if len(mid)]
    for cut in cuts:
        pairs, _ = ctx.pairlist(phi, g, cut)
        np.testing.assert_array_equal(pairs.cpu().numpy(), every[~off | (O >= cut)])
    # budget rule
    x = ctx.pair_features(phi, g)
    model = ctx.mlp_init(3)
    t = torch.linspace(-9.0, -2.0, max(2, len(iu)), device="cuda")
    ctx.mlp_fit_norm(model, x if len(iu) > 1 else x.repeat(2, 1), t)
    pred = ctx.mlp_forward(model, x, clamp=True).cpu().numpy()
    v = np.sort(pred[off])
    cum = np.cumsum(10.0 ** v.astype(np.float64))
    # budget -> smallest prediction that is kept
    cases = [(0.0, v[0] if off.any() else 0.0), (1e300, np.inf)]
    for f in (0.01, 0.2, 0.5, 0.9):
        k = int(f * len(v))
        if 0 < k < len(v) and v[k - 1] < v[k]:
            cases.append((0.5 * (cum[k - 1] + cum[k]), v[k]))
    if off.any():
        cases += [(1.001 * cum[-1], np.inf), (0.999 * (cum[-2] if len(cum) > 1 else cum[0]) + 0.0005 * 10.0 ** v[-1], None)]
    for budget, least in cases:
        if least is None:
            least = v[np.searchsorted(cum, budget, side="right")]
        pairs, fallback = ctx.screen_learned(phi, g, model, budget, 1e-3, 1e30)
        assert not fallback
        np.testing.assert_array_equal(pairs.cpu().numpy(), every[~off | (pred >= least)])


@pytest.mark.parametrize("n,stride", [(8, 1), (12, 3), (64, 2), (80, 5), (100, 2), (160, 4)])
def test_features(lib, n, stride):
    from paper_2101_03155_amd import Grid
    print(f"[gpu-case] features N={n} stride={stride}", flush=True)
    L, norb = 9.0, 3
    ctx, g = lib.Context(), Grid.cubic(n, L)
    r = np.arange(n) * L / n
    phi = np.empty((norb, n, n, n))
    for o, c in enumerate(((1.0, 4.0, 8.5), (4.4, 4.6, 1.0), (7.0, 0.5, 5.0))):
        d = [(r - x + L / 2) % L - L / 2 for x in c]
        # axes (z, y, x)
        phi[o] = np.exp(-0.5 * (d[2][:, None, None] ** 2 + d[1][None, :, None] ** 2 + d[0][None, None, :] ** 2))
    iu, ju = np.triu_indices(norb)
    f = ctx.pair_features(torch.as_tensor(phi, device="cuda"), g, stride=stride).cpu().numpy()
    ref = so.pair_features(phi, L, np.stack([iu, ju], 1), stride=stride)
    np.testing.assert_allclose(f[:, 0], ref[:, 0], atol=2e-6 * L)
    np.testing.assert_allclose(f[:, 1:3], ref[:, 1:3], rtol=2e-6)
    np.testing.assert_allclose(f[:, 3:], ref[:, 3:], atol=2e-5)
