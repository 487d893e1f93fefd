"""1D stages on systems whose sizes straddle every tile edge, in each launch
shape, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import step1d  # noqa: E402
from oracle.model import Params  # noqa: E402
from parity import check  # noqa: E402

pytestmark = pytest.mark.gpu

E = None
DX = 1 / 8
REACH = {8: 4.144547186125894, 16: 6.630878198393129, 24: 8.507803172628806}  # about the fastest velocity


def setup_module(module):
    global E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15187_amd import evlb as _E
    E = _E


def td(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


def moving_state(N, tb):
    """A state with flow, temperature and non-Maxwellian parts."""
    x = np.arange(N) / N
    F, G = step1d.initial_state(0.3 * (1 + 0.08 * np.sin(2 * np.pi * x + 0.1 * N)), 0.04 * np.cos(2 * np.pi * x),
                                0.6 + 0.02 * np.sin(2 * np.pi * x), tb)
    w = tb.w[:, None] / tb.w.max()
    bump = 1 + 0.03 * w * np.sin(0.37 * np.arange(N) + 1.3 * np.arange(len(tb.w))[:, None])
    return F * bump, G * bump[::-1]


# Sizes about the tiles of 16, 32 and 63 nodes.  tile 0 leaves the choice to
# the library: one copy of the sizes gives fewer tiles than CUs (narrow),
# twelve copies 516 narrow tiles (broad at q 8 and 16), and 70 1330 column
# tiles (column).
SIZES = (8, 9, 15, 16, 17, 30, 31, 32, 33, 47, 62, 63, 64, 65, 127)
EV1, EV2, NONE = 0, 1, 2


@pytest.mark.parametrize("Q", [8, 16, 24])
@pytest.mark.parametrize("tile,copies", [(16, 1), (63, 1), (64, 1), (0, 1), (0, 12), (0, 70)])
@pytest.mark.parametrize("force,mask,T_iso", [(EV1, 15, 0.0), (EV2, 15, 0.55), (NONE, 13, 0.0), (EV1, 14, 0.0)])
def test_tile_edges(Q, tile, copies, force, mask, T_iso):
    print(f"1D shape Q={Q} tile={tile} copies={copies} force={force} mask={mask} T_iso={T_iso}", flush=True)
    dt = 0.2 * DX / REACH[Q]
    kw = dict(force_model=force, term_mask=mask, T_iso=T_iso)
    tb = step1d.Tables(Params(Q=Q, dx=DX, dt=dt, **kw))
    states = [moving_state(N, tb) for N in SIZES]
    f0 = np.concatenate([np.stack(x) for x in states] * copies, axis=2)
    s = E.Solver(Q, DX, dt, list(SIZES) * copies, exec_mode=1, tile_nodes=tile, **kw)
    f = td(f0)
    L = s.rhs(f).cpu().numpy()
    s.step(f, 2)
    got = f.cpu().numpy()
    assert s.status() == 0
    total = sum(SIZES)
    for a in (L, got):  # equal systems give equal results wherever they lie
        for i in range(1, copies):
            assert np.array_equal(a[:, :, i * total:(i + 1) * total], a[:, :, :total])
    off = 0
    for N, (F, G) in zip(SIZES, states):
        check(L[:, :, off:off + N], step1d.rhs(F, G, tb), 1e-11, what=f"rhs {N}")
        check(got[:, :, off:off + N], step1d.run(F, G, tb, 2), 1e-11, steps=2, what=f"steps {N}")
        off += N


# every term by itself, and none, in the broad shape (one term at a time is
# tested elsewhere for the others)
@pytest.mark.parametrize("mask", [0, 1, 2, 4, 8])
@pytest.mark.parametrize("cells,r_cut", [(8, 5.0), (16, 4.0), (2, 1.0)])
def test_broad_terms_and_windows(mask, cells, r_cut):
    """cells = sigma/dx: 16 with r_cut = 4 sigma the widest windows, 2 with
    r_cut = sigma the narrowest."""
    print(f"1D broad mask={mask} cells={cells} r_cut={r_cut}", flush=True)
    dx = 1 / cells
    dt = 0.2 * dx / REACH[16]
    kw = dict(term_mask=mask, r_cut=r_cut)
    tb = step1d.Tables(Params(Q=16, dx=dx, dt=dt, **kw))
    nxs = [300] + [40] * 100
    states = {N: moving_state(N, tb) for N in set(nxs)}
    s = E.Solver(16, dx, dt, nxs, exec_mode=1, **kw)
    L = s.rhs(td(np.concatenate([np.stack(states[N]) for N in nxs], axis=2))).cpu().numpy()
    for off, N in ((0, 300), (300, 40), (300 + 99 * 40, 40)):
        ref = step1d.rhs(*states[N], tb)
        if mask == 0:
            assert not np.any(L)
        else:
            check(L[:, :, off:off + N], ref, 1e-11, what=f"{N} at {off}")


# 512 nodes are the last grid kept on one XCD (32 tiles on 256 CUs), 513 the
# first beyond it; 9 and 16: one tile
@pytest.mark.parametrize("N", [9, 16, 500, 512, 513, 530])
def test_one_xcd(N):
    print(f"1D one XCD N={N}", flush=True)
    dt = 0.2 * DX / REACH[16]
    tb = step1d.Tables(Params(Q=16, dx=DX, dt=dt))
    F, G = moving_state(N, tb)
    s = E.Solver(16, DX, dt, N)
    f = td(np.stack([F, G]))
    ref = step1d.moments(F, G, tb)
    got = s.moments(f).cpu().numpy()
    for i in range(4):
        assert np.max(np.abs(got[i] - ref[i])) <= 1e-13 * np.max(np.abs(ref[i])) + 1e-16, i
    s.step(f, 2)
    check(f.cpu().numpy(), step1d.run(F, G, tb, 2), 1e-11, steps=2, what=str(N))
    assert s.status() == 0
