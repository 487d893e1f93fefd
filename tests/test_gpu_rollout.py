"""Gradients of a rollout from its kept record against those from checkpoints,
in one, two and more segments with a short last one; which of the two ran is
read off the graph node."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

E = AD = None


def setup_module(module):
    global E, AD
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15187_amd import evlb as _E, adjoint as _AD
    E, AD = _E, _AD


def gradients(s, nsteps, every):
    x = torch.arange(s.n_tot, device="cuda", dtype=torch.float64) * (2 * torch.pi / s.n_tot)
    f0 = s.equilibrium(0.3 * (1 + 0.1 * torch.sin(x)), 0.05 * torch.cos(x), 0.6 + 0.02 * torch.sin(2 * x))
    f0.requires_grad_(True)
    par = [torch.ones((), device="cuda", dtype=torch.float64, requires_grad=True) for _ in range(2)]
    f, flux = AD.rollout(f0, *par, s, nsteps, 40, every)
    w = torch.sin(torch.arange(f.numel(), device="cuda", dtype=torch.float64)).view(f.shape)
    L = (w * f).sum() + (flux * torch.arange(1, nsteps + 1, device="cuda")).sum()
    return f.grad_fn, [f.detach(), flux.detach(), *torch.autograd.grad(L, [f0, *par])]


@pytest.mark.parametrize("nsteps,every,segments", [(1, 1, 1), (2, 2, 1), (2, 1, 2), (7, 4, 2), (9, 4, 3), (10, 3, 4)])
def test_record_and_checkpoints(nsteps, every, segments):
    print(f"rollout nsteps={nsteps} every={every}", flush=True)
    dx = 1 / 4
    s = E.Solver(16, dx, 0.2 * dx / 6.7, 150, adjoint=1)
    node, kept = gradients(s, nsteps, None)
    assert node.rec is not None and not node.ckpt
    node, again = gradients(s, nsteps, every)
    assert node.rec is None and len(node.ckpt) == segments
    for a, b in zip(kept, again):  # the same states are transposed; only sums may differ in order
        assert float((a - b).abs().max()) <= 1e-12 * float(b.abs().max())


def test_limit_of_no_bytes_takes_checkpoints(monkeypatch):
    dx = 1 / 4
    s = E.Solver(8, dx, 0.2 * dx / 6.7, 60, adjoint=1)
    monkeypatch.setattr(AD, "RECORD_BYTES", 0)
    for nsteps, segments in ((1, 1), (2, 1), (9, 3)):
        node, _ = gradients(s, nsteps, None)
        assert node.rec is None and len(node.ckpt) == segments
