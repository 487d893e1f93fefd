"""States, adjoint states and node fields that start on an odd multiple of eight
bytes: every entry point returns what it returns for arrays of the allocator's
alignment, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

E = None


def setup_module(module):
    global E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15187_amd import evlb as _E
    E = _E


def placed(x, odd):
    """A copy of x that starts one element into a buffer (odd) or at its start."""
    b = torch.empty(x.numel() + 1, dtype=torch.float64, device="cuda")
    y = b[odd:odd + x.numel()].view(x.shape)
    y.copy_(x)
    assert y.data_ptr() % 16 == 8 * odd
    return y


def fields(n_tot, dim):
    x = torch.arange(n_tot, device="cuda", dtype=torch.float64) * (2 * np.pi / n_tot)
    u = 0.05 * torch.cos(2 * x)
    return 0.3 * (1 + 0.1 * torch.sin(3 * x)), torch.stack([u, -u]) if dim == 2 else u, 0.6 + 0.02 * torch.sin(x)


def outputs(s, odd, adjoint):
    """What each entry point writes, all arrays placed alike."""
    new = lambda *shape: placed(torch.zeros(shape, dtype=torch.float64, device="cuda"), odd)
    n, u, T = (placed(x, odd) for x in fields(s.n_tot, s.dim))
    f = new(*s.new_state().shape)
    E.evlb_set_equilibrium(s.ctx, n, u, T, f)
    out = [f.clone()]
    L = new(*f.shape)
    E.evlb_rhs(s.ctx, f, L)
    E.evlb_step(s.ctx, f, 2)
    m = [new(*x.shape) for x in (n, u, T, u)]
    E.evlb_moments(s.ctx, f, *m)
    out += [L, f, *m]
    if adjoint:
        lam, par, rec = new(*f.shape), new(2), new(2 * s.record_doubles())
        E.evlb_adjoint_step(s.ctx, f, placed(L, odd), lam, par)
        E.evlb_step_record(s.ctx, f, 1, rec)
        back = placed(L, odd)
        E.evlb_adjoint_record(s.ctx, rec, 1, back, placed(f, odd), placed(torch.ones(1, device="cuda", dtype=torch.float64), odd), par)
        bars = [new(*x.shape) for x in (n, n, n)]
        E.evlb_equilibrium_adjoint(s.ctx, n, u, T, lam, *bars)
        out += [lam, par, rec[:s.record_doubles()], back, *bars]
    assert s.status() == 0
    return out


@pytest.mark.parametrize("kw", [dict(q=8, nx=100), dict(q=16, nx=6000), dict(q=24, nx=[130, 61]),
                                dict(q=16, nx=50000, tile_nodes=64), dict(q=16, nx=3000, tile_nodes=63),
                                dict(q=16, nx=33, ny=21)])
def test_eight_byte_alignment(kw):
    print(f"alignment {kw}", flush=True)
    dx = 1 / 4 if "ny" in kw else 1 / 8
    adjoint = "ny" not in kw
    kw = dict(kw)
    s = E.Solver(kw.pop("q"), dx, 0.2 * dx / 8.6, kw.pop("nx"), adjoint=int(adjoint), **kw)
    for a, b in zip(outputs(s, 0, adjoint), outputs(s, 1, adjoint)):
        assert torch.equal(a, b)
