"""The persistent launch on grids of more tiles than CUs: the steps of the
per-stage launches, and a clean status (a barrier that times out latches one)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from parity import check  # noqa: E402

pytestmark = pytest.mark.gpu

E = None


def setup_module(module):
    global E
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_15187_amd import evlb as _E
    E = _E


# tiles of 16 nodes: 513 and 1100 of them (more than two and four per CU), in
# one system and in two, with all terms and with some; 63 and 64: more than four
# per CU
@pytest.mark.parametrize("Q", [8, 16, 24])
@pytest.mark.parametrize("tile,nx,mask", [(16, [8200], 15), (16, [9000, 8600], 15), (16, [9000, 8600], 5),
                                          (63, [65000], 15), (64, [70000], 15)])
def test_more_tiles_than_compute_units(Q, tile, nx, mask):
    print(f"persistent Q={Q} tile={tile} nx={nx} mask={mask}", flush=True)
    dx = 1 / 8
    dt = 0.2 * dx / 8.6
    out = []
    for mode in (E.EVLB_EXEC_PER_STAGE, E.EVLB_EXEC_PERSISTENT):
        s = E.Solver(Q, dx, dt, nx, exec_mode=mode, tile_nodes=tile, term_mask=mask)
        x = torch.arange(s.n_tot, device="cuda", dtype=torch.float64) * (2 * np.pi / s.n_tot)
        f = s.equilibrium(0.3 * (1 + 0.1 * torch.sin(40 * x)), 0.05 * torch.cos(30 * x), 0.6 + 0.02 * torch.sin(x))
        s.step(f, 3)
        assert s.status() == 0
        out.append(f.cpu().numpy())
    check(out[1], out[0], 1e-11, steps=3, what=f"{Q} {tile}")
