"""The adjoint of a step on systems whose sizes straddle the edges of its tiles
(16 and 59 nodes), and at the widest and narrowest windows: dot products with
complex-step derivatives of the oracle's step, per system, and the parameter
derivatives."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import step1d  # noqa: E402
from oracle.model import Params  # noqa: E402

pytestmark = pytest.mark.gpu

E = None
H = 1e-30
EV1, NONE = 0, 2


def setup_module(module):
    global E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15187_amd import evlb as _E
    E = _E


def td(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


SIZES = (8, 9, 15, 16, 17, 31, 33, 58, 59, 60, 64, 65, 118, 119)


@pytest.mark.parametrize("Q", [8, 16, 24])
@pytest.mark.parametrize("cells,r_cut,force,mask", [(8, 5.0, EV1, 15), (16, 4.0, EV1, 15), (2, 1.0, EV1, 15),
                                                    (8, 5.0, NONE, 13), (4, 5.0, EV1, 6), (4, 5.0, EV1, 11)])
def test_tile_edges_dot_product(Q, cells, r_cut, force, mask):
    print(f"adjoint shape Q={Q} cells={cells} r_cut={r_cut} force={force} mask={mask}", flush=True)
    dx = 1 / cells
    dt = 0.2 * dx / 8.6
    kw = dict(r_cut=r_cut, force_model=force, term_mask=mask)
    tb = step1d.Tables(Params(Q=Q, dx=dx, dt=dt, **kw))
    rng = np.random.default_rng(100 * Q + cells)
    fs, vs, lams = [], [], []
    for N in SIZES:
        x = np.arange(N) / N
        F, G = step1d.initial_state(0.3 * (1 + 0.1 * np.sin(2 * np.pi * x + N)), 0.05 * np.cos(2 * np.pi * x),
                                    0.6 * (1 + 0.05 * np.sin(2 * np.pi * x)), tb)
        f = np.stack([F, G]) * (1 + 0.03 * rng.standard_normal((2, Q, N)))
        fs.append(f)
        vs.append(rng.standard_normal((2, Q, N)) * f)
        lams.append(rng.standard_normal((2, Q, N)))
    s = E.Solver(Q, dx, dt, list(SIZES), adjoint=1, **kw)
    dpar = torch.zeros(2, dtype=torch.float64, device="cuda")
    got = s.adjoint_step(td(np.concatenate(fs, axis=2)), td(np.concatenate(lams, axis=2)), dpar).cpu().numpy()
    off = 0
    for N, f, v, lam in zip(SIZES, fs, vs, lams):
        F1, G1 = step1d.rk3_step(f[0] + 1j * H * v[0], f[1] + 1j * H * v[1], tb)
        ref = (np.sum(lam[0] * F1) + np.sum(lam[1] * G1)).imag / H
        g = got[:, :, off:off + N]
        # rounding of the two sums: a few ulp of the sum of magnitudes
        assert abs(np.sum(g * v) - ref) <= 1e-12 * np.sum(np.abs(g * v)), (N, np.sum(g * v), ref)
        off += N
    for i, which in enumerate(("phi", "sigma")):
        tc = step1d.Tables(Params(Q=Q, dx=dx, dt=dt, **{which: 1.0 + 1j * H}, **kw))
        ref = 0.0
        for f, lam in zip(fs, lams):
            F1, G1 = step1d.rk3_step(f[0].astype(complex), f[1].astype(complex), tc)
            ref += (np.sum(lam[0] * F1) + np.sum(lam[1] * G1)).imag / H
        assert abs(float(dpar[i]) - ref) <= 1e-10 * max(1.0, abs(ref)), (which, float(dpar[i]), ref)


@pytest.mark.parametrize("nsteps", [1, 2, 9])
def test_kept_record_and_checkpoints_agree(nsteps, monkeypatch):
    """The rollout's gradients from its kept record, and from checkpoints (a
    limit of no bytes): the same states are transposed, so only the order of
    the parameter sums and of the flux product may differ; and a second
    backward pass over the same graph repeats the first."""
    from paper_2503_15187_amd import adjoint as AD
    print(f"rollout record nsteps={nsteps}", flush=True)
    N, dx = 150, 1 / 4
    dt = 0.2 * dx / 6.7
    s = E.Solver(16, dx, dt, N, adjoint=1)
    x = torch.arange(N, device="cuda", dtype=torch.float64) / N
    out = []
    for limit in (AD.RECORD_BYTES, 0):
        monkeypatch.setattr(AD, "RECORD_BYTES", limit)
        n0 = (0.3 * (1 + 0.1 * torch.sin(2 * np.pi * x))).requires_grad_(True)
        par = [torch.ones((), device="cuda", dtype=torch.float64, requires_grad=True) for _ in range(2)]
        L = AD.slab_loss(n0, *par, s, nsteps, 40, dt, dx, 0.3 + 0 * x, 0.6 + 0 * x)
        g = torch.autograd.grad(L, [n0, *par], retain_graph=True)
        for a, b in zip(g, torch.autograd.grad(L, [n0, *par])):
            assert torch.equal(a, b)
        out.append([L.detach(), *g])
    for a, b in zip(*out):
        assert float((a - b).abs().max()) <= 1e-12 * float(b.abs().max())
