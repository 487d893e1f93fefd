"""2D steps on the smallest grids and on grids whose strips and segments of
rows fall unevenly on the CUs, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
from oracle import step2d  # noqa: E402
from oracle.model import Params  # noqa: E402
from parity import check  # noqa: E402

pytestmark = pytest.mark.gpu

E = None


def setup_module(module):
    global E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15187_amd import evlb as _E
    E = _E


def td(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def moving_state(nx, ny, tb):
    """A state with flow, temperature and non-Maxwellian parts."""
    c, n, ux, uy, T = workloads.phase_separation_2d(nx=nx, ny=ny)
    yy, xx = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
    ux = 0.03 * np.sin(2 * np.pi * xx / nx) * np.cos(2 * np.pi * yy / ny)
    uy = -0.02 * np.cos(4 * np.pi * xx / nx)
    T = T * (1 + 0.02 * np.sin(2 * np.pi * yy / ny))
    F, G = step2d.initial_state(n, ux, uy, T, tb)
    w = tb.w / tb.w.max()
    k, l = np.arange(16)[:, None, None, None], np.arange(16)[None, :, None, None]
    bump = 1 + 0.03 * w[:, None, None, None] * w[None, :, None, None] * np.sin(0.37 * xx + 0.61 * yy + 1.3 * k + 0.7 * l)
    return F * bump, G * bump[:, ::-1]


# (8, 8): one strip, one row per segment; (16, 11): segments of one row, an odd
# number of rows; (130, 17): a two-column last strip; (200, 26): 50 strips and
# distributions in segments of 6 and 2 rows; (1032, 8): more strips than CUs,
# two rounds
@pytest.mark.parametrize("nx,ny,nsteps", [(8, 8, 2), (16, 11, 2), (130, 17, 1), (200, 26, 1), (1032, 8, 1)])
def test_steps_match_oracle(nx, ny, nsteps):
    print(f"2D shape nx={nx} ny={ny} nsteps={nsteps}", flush=True)
    c = workloads.constants()["phase_separation_2d"]
    tb = step2d.Tables2D(Params(Q=16, dx=c["dx"], dt=c["dt"]))
    F, G = moving_state(nx, ny, tb)
    s = E.Solver(16, c["dx"], c["dt"], nx, ny=ny)
    f = E.Solver.from_planes(td(np.stack([F, G])))
    s.step(f, nsteps)
    torch.cuda.synchronize()
    F, G = step2d.run(F, G, tb, nsteps)
    check(E.Solver.planes(f).cpu().numpy(), [F, G], 1e-11, steps=nsteps, what=f"{nx}x{ny}")
    assert s.status() == 0


# the widest stencils the parameters admit (averaging radius 22 cells, force
# radius 24 or 23) and narrow ones (averaging disc of one cell, force radius 1)
@pytest.mark.parametrize("cells,reach", [(22.0, 24), (21.5, 23), (0.9, 1), (2.0, 3)])
def test_rhs_stencil_widths(cells, reach):
    print(f"2D stencils sigma/dx={cells} r_cut/dx={reach}", flush=True)
    nx, ny, dx = 40, 27, 1.0 / cells
    p = dict(dx=dx, dt=0.2 * dx / 6.630878198393129, r_cut=reach * dx)
    tb = step2d.Tables2D(Params(Q=16, **p))
    F, G = moving_state(nx, ny, tb)
    s = E.Solver(16, p["dx"], p["dt"], nx, ny=ny, r_cut=p["r_cut"])
    L = E.Solver.planes(s.rhs(E.Solver.from_planes(td(np.stack([F, G])))))
    torch.cuda.synchronize()
    check(L.cpu().numpy(), step2d.rhs(F, G, tb), 1e-11, what=f"{cells} {reach}")
    assert s.status() == 0


# node counts around the 16 and 32 nodes a workgroup takes, and one past both
@pytest.mark.parametrize("nx,ny", [(8, 8), (9, 11), (33, 31), (8, 9)])
@pytest.mark.parametrize("heat", [True, False])
def test_equilibrium_and_moments_match_oracle(nx, ny, heat):
    print(f"2D observe nx={nx} ny={ny} heat={heat}", flush=True)
    c = workloads.constants()["phase_separation_2d"]
    tb = step2d.Tables2D(Params(Q=16, dx=c["dx"], dt=c["dt"]))
    rng = np.random.default_rng(nx * ny)
    n, T = (b * (1 + 0.1 * rng.standard_normal((ny, nx))) for b in (0.3, 0.6))
    u = 0.1 * rng.standard_normal((2, ny, nx))
    s = E.Solver(16, c["dx"], c["dt"], nx, ny=ny)
    f = s.equilibrium(td(n), td(u), td(T))
    ref = step2d.initial_state(n, u[0], u[1], T, tb)
    check(E.Solver.planes(f).cpu().numpy(), ref, 1e-11, what="equilibrium")
    F, G = moving_state(nx, ny, tb)
    g = E.Solver.from_planes(td(np.stack([F, G])))
    m = np.stack(step2d.moments(F, G, tb)).reshape(6, -1)
    out = torch.full((6, nx * ny), 7.0, dtype=torch.float64, device="cuda")
    E.evlb_moments(s.ctx, g, out[0], out[1:3], out[3], out[4:6] if heat else None)
    got = out.cpu().numpy()
    # sums of 512 terms with weights up to 6.7^3: a few hundred roundings of the largest moment
    assert np.max(np.abs(got[:4] - m[:4])) < 1e-12
    if heat:
        assert np.max(np.abs(got[4:] - m[4:])) < 1e-12
    else:
        assert np.all(got[4:] == 7.0)
