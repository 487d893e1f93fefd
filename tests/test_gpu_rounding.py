"""Rounding of one step against the oracle in extended precision (the same double
constants): how many roundings of the size of the result a stage makes.

A rounding of x to double has an rms of 4.7e-17 |x| (uniform within half a unit,
x spread evenly in its logarithm).  A stage that sums c L(f) first and then adds
b f^(s-1) and a f^n rounds once at b f and once at f; over the three stages of a
step (b = 1, 1/4, 2/3) that is 6.5e-17.  The 2D stage adds two terms of L behind
these: 1.05e-16.  The bars leave 1.3 and 1.25 of these for the rounding of L;
the terms of L added to the states one by one gave 9.4 to 10e-17 and 1.5e-16."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads  # noqa: E402
from oracle import step1d, step2d  # noqa: E402
from oracle.model import Params  # noqa: E402

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


def rms(got, ref):
    """rms relative error over the values above 1e-3 of the largest."""
    big = np.abs(ref) > 1e-3 * np.abs(ref).max()
    return float(np.sqrt(np.mean(((got - ref)[big] / ref[big]) ** 2)))


needs_extended = pytest.mark.skipif(np.finfo(np.longdouble).nmant <= 52, reason="no extended precision")


@needs_extended
@pytest.mark.parametrize("Q,reach", [(8, 4.144547186125894), (16, 6.630878198393129), (24, 8.507803172628806)])
@pytest.mark.parametrize("tile", [63, 64])
def test_step_1d(Q, reach, tile):
    N, dx = 504, 1 / 8
    dt = 0.2 * dx / reach
    tb = step1d.Tables(Params(Q=Q, dx=dx, dt=dt))
    x = np.arange(N) / N
    noise = 0.01 * np.random.default_rng(Q).standard_normal(N)
    F, G = step1d.initial_state(0.3 * (1 + 0.08 * np.sin(2 * np.pi * x) + noise), 0.04 * np.cos(2 * np.pi * x),
                                0.6 + 0.02 * np.sin(2 * np.pi * x), tb)
    s = E.Solver(Q, dx, dt, N, exec_mode=1, tile_nodes=tile)
    f = td(np.stack([F, G]))
    s.step(f, 1)
    ref = np.stack(step1d.run(F.astype(np.longdouble), G.astype(np.longdouble), tb, 1))
    assert ref.dtype == np.longdouble
    e = rms(f.cpu().numpy(), ref)
    print(f"Q={Q} tile={tile} rms {e:.2e}", flush=True)
    assert e <= 1.3 * 6.5e-17


@needs_extended
def test_step_2d():
    nx, ny = 40, 24
    c, n, ux, uy, T = workloads.phase_separation_2d(nx=nx, ny=ny)
    yy, xx = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
    tb = step2d.Tables2D(Params(Q=16, dx=c["dx"], dt=c["dt"]))
    F, G = step2d.initial_state(n, 0.03 * np.sin(2 * np.pi * xx / nx), -0.02 * np.cos(2 * np.pi * yy / ny), T, tb)
    s = E.Solver(16, c["dx"], c["dt"], nx, ny=ny)
    f = E.Solver.from_planes(td(np.stack([F, G])))
    s.step(f, 1)
    ref = np.stack(step2d.run(F.astype(np.longdouble), G.astype(np.longdouble), tb, 1))
    assert ref.dtype == np.longdouble
    e = rms(E.Solver.planes(f).cpu().numpy(), ref)
    print(f"2D rms {e:.2e}", flush=True)
    assert e <= 1.25 * 1.05e-16
