"""What a rollout keeps for its backward pass, decided on the host: the record,
checkpoints or nothing.  The solver is a stand-in whose step adds one."""
import pytest

torch = pytest.importorskip("torch")

from paper_2503_15187_amd import adjoint as AD  # noqa: E402


class Counter:
    """record layout of Solver: states of 2 q n_tot values, R values a record"""
    q, n_tot, velocities = 2, 3, [-1.0, 1.0]

    def __init__(self):
        self.largest = 0

    def record_doubles(self):
        return 20

    def record_buffer(self, nsteps):
        self.largest = max(self.largest, nsteps)
        return torch.zeros((nsteps + 1) * 20, dtype=torch.float64)

    def record_state(self, rec, j):
        return rec[20 * j:20 * j + 12].view(2, 2, 3)

    def step_record(self, f0, nsteps, rec):
        for j in range(nsteps + 1):
            self.record_state(rec, j).copy_(f0 + j)


@pytest.fixture
def memory(monkeypatch):
    """Sets the device's free bytes and the record limit."""
    def set_(free, limit):
        monkeypatch.setattr(torch.cuda, "mem_get_info", lambda device=None: (free, free))
        monkeypatch.setattr(AD, "RECORD_BYTES", limit)
    return set_


def run(nsteps, grad=True, every=None, solver=None):
    s = solver or Counter()
    f0 = torch.zeros((2, 2, 3), dtype=torch.float64, requires_grad=grad)
    one = torch.ones((), dtype=torch.float64)
    f, flux = AD.rollout(f0, one, one.clone(), s, nsteps, 1, every)
    assert torch.equal(f, torch.full_like(f, float(nsteps)))
    assert flux.shape == (nsteps,) and not flux.any()  # sum of p F, F equal at both velocities
    return s, f.grad_fn


@pytest.mark.parametrize("nsteps,starts", [(1, [0]), (2, [0]), (3, [0, 2]), (9, [0, 3, 6]), (10, [0, 4, 8])])
@pytest.mark.parametrize("free,limit", [(1 << 40, 0), (0, 1 << 30)])
def test_checkpoints_where_the_record_is_too_large(memory, nsteps, starts, free, limit):
    memory(free, limit)
    s, node = run(nsteps)
    assert node.rec is None and sorted(node.ckpt) == starts
    assert s.largest == AD.checkpoint_steps(nsteps) == AD.segment_steps(s, nsteps, None)
    assert not AD.keeps_record(s, nsteps, None)


@pytest.mark.parametrize("nsteps", [1, 2, 3, 10])
def test_record_where_it_fits(memory, nsteps):
    memory(1 << 40, 1 << 30)
    s, node = run(nsteps)
    assert node.rec is not None and not node.ckpt and s.largest == nsteps
    memory(32 * 8 * 20 * (nsteps + 1), 8 * 20 * (nsteps + 1))  # just fits
    assert AD.keeps_record(s, nsteps, None)
    memory(32 * 8 * 20 * (nsteps + 1) - 1, 8 * 20 * (nsteps + 1))
    assert not AD.keeps_record(s, nsteps, None)


@pytest.mark.parametrize("every,starts", [(1, [0, 1, 2, 3]), (3, [0, 3]), (4, [0]), (7, [0])])
def test_given_segments_are_taken(memory, every, starts):
    memory(1 << 40, 1 << 30)
    _, node = run(4, every=every)
    assert node.rec is None and sorted(node.ckpt) == starts


def test_nothing_is_kept_without_a_gradient(memory):
    memory(1 << 40, 1 << 30)
    s, node = run(100, grad=False)
    assert node is None and s.largest == 10
    s = Counter()
    with torch.no_grad():
        _, node = run(100, solver=s)
    assert node is None and s.largest == 10


def test_no_steps(memory):
    memory(1 << 40, 1 << 30)
    s, node = run(0)
    assert node.rec is None and not node.ckpt
