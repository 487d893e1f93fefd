"""The autotuner's candidates and its cache, with a stand-in solver and clock."""
import json

import pytest

torch = pytest.importorskip("torch")

from paper_2503_15187_amd import autotune as AT, evlb as E  # noqa: E402

LIBRARY, NARROW, COLUMN = (E.EVLB_EXEC_PER_STAGE, 0), (E.EVLB_EXEC_PER_STAGE, 16), (E.EVLB_EXEC_PER_STAGE, 63)


@pytest.fixture
def tuner(monkeypatch, tmp_path):
    """tune() over stand-in solvers: a step takes the seconds that `cost` gives
    its candidate (1 if none), on a clock of its own."""
    class State:
        cost, now, build, device = {}, 0.0, "a", "card 1"

    class Solver:
        def __init__(self, q, dx, dt, nx, device=None, exec_mode=0, tile_nodes=0, **kw):
            self.key = (exec_mode, tile_nodes)

        def step(self, f, n):
            State.now += n * State.cost.get(self.key, 1.0)

        def status(self):
            return 0

    monkeypatch.setattr(E, "Solver", Solver)
    monkeypatch.setattr(AT, "_CACHE_PATH", str(tmp_path / "tune.json"))
    monkeypatch.setattr(AT, "_memo", {})
    monkeypatch.setattr(AT, "_build_id", lambda: State.build)
    monkeypatch.setattr(AT.time, "perf_counter", lambda: State.now)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda device=None: State.device)

    def tune(nx=1000, dx=0.125, **kw):
        mode, tile, _ = AT.tune(16, dx, 1e-3, nx, torch.zeros(2), **kw)
        return mode, tile
    return State, tune


def test_the_librarys_own_choice_can_win(tuner):
    state, tune = tuner
    state.cost = {LIBRARY: 0.5}
    assert tune() == LIBRARY
    state.cost = {LIBRARY: 0.5, COLUMN: 0.4}
    assert tune(nx=2000) == COLUMN


@pytest.mark.parametrize("change", [dict(build="b"), dict(device="card 2"), dict(dx=0.25), dict(r_cut=4.0),
                                    dict(T_iso=0.6), dict(T_iso_sys=[0.6]), dict(term_mask=5), dict(nx=1001)])
def test_a_winner_holds_for_its_problem_build_and_device(tuner, change):
    state, tune = tuner
    state.cost = {NARROW: 0.5}
    assert tune() == NARROW
    state.cost = {COLUMN: 0.5}
    assert tune() == NARROW  # from the cache
    AT._memo.clear()
    assert tune() == NARROW  # and from its file
    kw = dict(change)
    for name in ("build", "device"):
        if name in kw:
            setattr(state, name, kw.pop(name))
    assert tune(**kw) == COLUMN


def test_entries_without_a_build_are_not_taken(tuner, tmp_path):
    """A file written before the signature named the build."""
    state, tune = tuner
    (tmp_path / "tune.json").write_text(json.dumps({AT.signature(16, 1000): [*NARROW, 1e-6]}))
    state.cost = {COLUMN: 0.5}
    assert tune() == COLUMN


def test_the_build_id_is_the_librarys(tmp_path, monkeypatch):
    monkeypatch.setattr(E, "LIB_PATH", str(tmp_path / "lib.so"))
    ids = []
    for text in ("one", "two"):
        (tmp_path / "lib.so").write_text(text)
        ids.append(AT._build_id.__wrapped__())
    assert ids[0] != ids[1]
