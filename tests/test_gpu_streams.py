"""Several contexts in flight on streams of their own, small grids that share one
XCD among them: each returns what it returns alone, bit for bit."""
import threading

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


# grids of at most 512 nodes run on one XCD; 600 and the 2D box do not
GRIDS = [dict(q=8, nx=500), dict(q=16, nx=512), dict(q=24, nx=[100, 333]), dict(q=16, nx=64), dict(q=16, nx=600),
         dict(q=16, nx=40, ny=24)]


def start(kw):
    kw = dict(kw)
    dx = 1 / 4 if "ny" in kw else 1 / 8
    s = E.Solver(kw.pop("q"), dx, 0.2 * dx / 8.6, kw.pop("nx"), adjoint=int("ny" not in kw), **kw)
    x = torch.arange(s.n_tot, device="cuda", dtype=torch.float64) * (2 * torch.pi / s.n_tot)
    u = 0.05 * torch.cos(x)
    f = s.equilibrium(0.3 * (1 + 0.1 * torch.sin(x)), torch.stack([u, u]) if s.dim == 2 else u, 0.6 + 0 * x)
    return s, f


def calls(s, f):
    """Steps, a right-hand side, moments and (1D) an adjoint step, as pieces to be interleaved."""
    out = [f]
    for _ in range(10):
        s.step(f, 3)
        yield out
    out += [s.rhs(f), s.moments(f)]
    yield out
    if s.dim == 1:
        par = torch.zeros(2, dtype=torch.float64, device="cuda")
        out += [s.adjoint_step(f, out[1], par), par]
        yield out


def last(it):
    for out in it:
        pass
    return out


def same(got, ref):
    assert len(got) == len(ref)
    for a, b in zip(got, ref):
        assert torch.equal(a, b)


def test_interleaved_on_streams():
    alone = [last(calls(*start(kw))) for kw in GRIDS]
    torch.cuda.synchronize()
    pairs = [start(kw) for kw in GRIDS]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in GRIDS]
    its = [calls(s, f) for s, f in pairs]
    results = [None] * len(GRIDS)
    while any(it is not None for it in its):
        for i, (it, st) in enumerate(zip(its, streams)):
            if it is None:
                continue
            with torch.cuda.stream(st):
                out = next(it, None)
            if out is None:
                its[i] = None
            else:
                results[i] = out
    torch.cuda.synchronize()
    for (s, _), got, ref in zip(pairs, results, alone):
        assert s.status() == 0
        same(got, ref)


def test_gradients_in_threads():
    """Rollouts with a kept record and with checkpoints, each thread on its own
    stream and solver."""
    def grads(every):
        s, f0 = start(dict(q=16, nx=300))
        f0.requires_grad_(True)
        par = [torch.ones((), device="cuda", dtype=torch.float64, requires_grad=True) for _ in range(2)]
        f, flux = AD.rollout(f0, *par, s, 12, 20, every)
        return list(torch.autograd.grad(f.square().sum() + flux.sum(), [f0, *par]))

    jobs = [None, 4, None, 5]
    alone = [grads(every) for every in jobs]
    torch.cuda.synchronize()
    got, streams = [None] * len(jobs), [torch.cuda.Stream() for _ in jobs]

    def work(i):
        with torch.cuda.stream(streams[i]):
            got[i] = grads(jobs[i])
            streams[i].synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, b in zip(got, alone):
        same(a, b)
