"""The screener's minibatch gradient against FP64 autograd at the edges of its
64-sample chunks, with a ragged last chunk, and where blocks take more than one
chunk (over 65536 samples).  Tolerance: FP32 products of 64 terms, tanh to a few
ulp and sums over at most 64 chunks in order, each rounding 6e-8 and mostly
independent: about 1e-6 of the gradient's 2-norm; 5e-6 is asserted."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _reference(model, x, t):
    from paper_2101_03155_amd import ace
    p = model[:ace.MLP_NPARAM].double().clone().requires_grad_(True)
    norm = model[ace.MLP_NPARAM:].double()
    xs = (x.double() - norm[:5]) / norm[5:10]
    ts = (t.double() - norm[10]) / norm[11]
    h = torch.tanh(xs @ p[:320].view(64, 5).T + p[320:384])
    h = torch.tanh(h @ p[384:4480].view(64, 64).T + p[4480:4544])
    loss = ((h @ p[4544:4608] + p[4608] - ts) ** 2).mean()
    g, = torch.autograd.grad(loss, p)
    return g, loss.detach()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 4096, 70001])
def test_gradient_against_autograd(lib, n):
    print(f"[gpu-case] screener gradient, {n} samples", flush=True)
    ctx = lib.Context()
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(n, 5, device="cuda", generator=g) * 2 + 1
    t = torch.randn(n, device="cuda", generator=g) - 2
    model = ctx.mlp_init(7)
    ctx.mlp_fit_norm(model, torch.randn(512, 5, device="cuda", generator=g) * 2 + 1,
                     torch.randn(512, device="cuda", generator=g) - 2)
    got, loss = ctx.mlp_grad(model, x, t)
    ref, ref_loss = _reference(model, x, t)
    err = float((got.double() - ref).norm() / ref.norm())
    print(f"  gradient rel err {err:.2e}, loss {loss.item():.8f} vs {ref_loss.item():.8f}", flush=True)
    assert err <= 5e-6
    assert abs(loss.item() - ref_loss.item()) <= 5e-6 * ref_loss.item()
    again, _ = ctx.mlp_grad(model, x, t)
    assert torch.equal(got, again)  # summed in a fixed order
