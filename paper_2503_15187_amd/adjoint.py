"""Differentiable EV-FDLB runs on top of the discrete-adjoint C ABI.

Rollout (a torch.autograd.Function) advances a state nsteps TVD-RK3 steps
and returns the final state together with the history of the mass flux
sum_k p_k F_k through one node after every step.  A run whose record (states
and stage states of every step) is small keeps it, and the backward pass
transposes it with evlb_adjoint_record; without a gradient to come nothing is
kept.  Of a larger one the forward pass
keeps a checkpoint every ceil(sqrt(nsteps)) steps; the backward pass re-runs
each segment from its checkpoint with evlb_step_record and transposes it,
walking the segments in reverse, the recomputation of the next segment on a
second context and stream overlapping the transposition of the current one.
It returns the gradients with respect to the initial state and to the
parameters phi_sigma and sigma (the latter two enter as 0-d tensors whose
values must equal the context's; they only carry the gradient).

Equilibrium maps (n, u, T) fields to the initial reduced Maxwellian with
evlb_set_equilibrium; its backward uses evlb_equilibrium_adjoint.
"""
import math

import torch


class Equilibrium(torch.autograd.Function):
    @staticmethod
    def forward(ctx, n, u, T, solver):
        ctx.solver = solver
        ctx.save_for_backward(n, u, T)
        return solver.equilibrium(n.detach().contiguous(), u.detach().contiguous(), T.detach().contiguous())

    @staticmethod
    def backward(ctx, lam):
        n, u, T = ctx.saved_tensors
        g = ctx.solver.equilibrium_adjoint(n.contiguous(), u.contiguous(), T.contiguous(), lam.contiguous())
        return g[0], g[1], g[2], None


# Largest record that a run keeps, if it is also at most 1/32 of the device's free
# memory (many runs may be alive at once: a graph holds its record as long as
# its outputs live).  Keeping it saves the recomputation, a third of the backward
# pass's launches.  It is faster at every size, so the line is what memory a
# graph may hold, not a crossover; what a longer run gives up for it:
#   gradient, record / checkpoints   64 steps           512              2000
#   2048 nodes  q 8                  2.9 / 4.2 ms    19.6 / 26.1    76 /  97 (1.9 GB)
#               q 16                 3.1 / 3.9       21.5 / 24.1    84 /  97 (3.5 GB)
#               q 24                 3.7 / 4.3       25.9 / 28.6   100 / 108 (5.1 GB)
RECORD_BYTES = 512 << 20


def keeps_record(solver, nsteps, device):
    """Whether a run of nsteps steps keeps its record for the backward pass."""
    nbytes = 8 * (nsteps + 1) * solver.record_doubles()
    return 0 < nsteps and nbytes <= RECORD_BYTES and 32 * nbytes <= torch.cuda.mem_get_info(device)[0]


def checkpoint_steps(nsteps):
    return max(1, int(math.ceil(math.sqrt(nsteps))))


def segment_steps(solver, nsteps, device):
    """Steps between checkpoints, unless the caller gives them: all of them
    if their record is small enough to be kept, else ceil(sqrt(nsteps))."""
    return nsteps if keeps_record(solver, nsteps, device) else checkpoint_steps(nsteps)


class Rollout(torch.autograd.Function):
    @staticmethod
    def forward(ctx, f0, phi, sigma, solver, nsteps, flux_node, every=None):
        nsteps = int(nsteps)
        dev = f0.device
        # without a gradient to come neither a record nor checkpoints are kept
        grad = any(ctx.needs_input_grad[:3])
        keep = grad and not every and keeps_record(solver, nsteps, dev)
        every = int(every) if every else (nsteps if keep else checkpoint_steps(nsteps))
        vel = torch.tensor(solver.velocities, dtype=torch.float64, device=dev)
        rec = solver.record_buffer(every)
        R = rec.numel() // (every + 1)
        N = solver.n_tot
        node = int(flux_node)
        f = f0.detach().contiguous()
        ckpt = {}
        flux = torch.empty(nsteps, dtype=torch.float64, device=dev)
        for start in range(0, nsteps, every):
            seg = min(every, nsteps - start)
            if grad and not keep:
                ckpt[start] = f.clone()
            solver.step_record(f, seg, rec)
            # F_k(node) of the states 1 .. seg inside the record, k = 0 .. q - 1
            flux[start:start + seg] = rec.as_strided((seg, solver.q), (R, N), R + node) @ vel
            f = solver.record_state(rec, seg).clone()
        ctx.solver, ctx.nsteps, ctx.every, ctx.flux_node = solver, nsteps, every, flux_node
        ctx.ckpt, ctx.rec, ctx.vel = ckpt, rec if keep else None, vel
        ctx.shape = f.shape
        return f, flux

    @staticmethod
    def backward(ctx, g_f, g_flux):
        solver, nsteps, every, node = ctx.solver, ctx.nsteps, ctx.every, ctx.flux_node
        lam = ctx.vel.new_zeros(ctx.shape) if g_f is None else g_f.detach().clone().contiguous()
        obs = w = None
        if g_flux is not None:
            obs = torch.zeros_like(lam)
            obs[0, :, node] = ctx.vel
            w = g_flux.detach().contiguous()
        dparams = torch.zeros(2, dtype=torch.float64, device=lam.device)
        if ctx.rec is not None:
            solver.adjoint_record(ctx.rec, nsteps, lam, dparams, obs, w)
            return lam, dparams[0], dparams[1], None, None, None, None
        # The segments in reverse.  The recomputation of segment i + 1 (a
        # second context on a second stream, into the other record buffer)
        # runs while segment i is transposed: the two chains of small
        # launches fill the device together.
        starts = sorted(ctx.ckpt, reverse=True)
        recomp = getattr(solver, "_adjoint_twin", None)
        if recomp is None:
            recomp = solver._adjoint_twin = solver.twin()
        recs = [solver.record_buffer(every), solver.record_buffer(every)]
        main = torch.cuda.current_stream(lam.device)
        side = torch.cuda.Stream(device=lam.device)
        side.wait_stream(main)
        ready = [torch.cuda.Event() for _ in starts]
        freed = [torch.cuda.Event(), torch.cuda.Event()]

        def recompute(i):
            seg = min(every, nsteps - starts[i])
            if i >= 2:
                side.wait_event(freed[i % 2])  # segment i - 2 no longer reads this buffer
            recomp.step_record(ctx.ckpt[starts[i]], seg, recs[i % 2], stream=side)
            ready[i].record(side)

        recompute(0)
        if len(starts) > 1:
            recompute(1)
        for i, start in enumerate(starts):
            seg = min(every, nsteps - start)
            main.wait_event(ready[i])
            solver.adjoint_record(recs[i % 2], seg, lam, dparams, obs, None if w is None else w[start:start + seg],
                                  stream=main)
            freed[i % 2].record(main)
            if i + 2 < len(starts):
                recompute(i + 2)
        for r in recs:
            r.record_stream(side)
        return lam, dparams[0], dparams[1], None, None, None, None


def rollout(f0, phi, sigma, solver, nsteps, flux_node, every=None):
    if not torch.is_grad_enabled():  # a Function sees its inputs' flags, not the mode
        f0, phi, sigma = (x.detach() if torch.is_tensor(x) else x for x in (f0, phi, sigma))
    return Rollout.apply(f0, phi, sigma, solver, nsteps, flux_node, every)


def slab_loss(n0, phi, sigma, solver, nsteps, flux_node, dt, dx, target, T0, every=None):
    """Time-integrated mass flux through flux_node plus the L2 misfit of the
    final density to a target: L = dt sum_n J(f^n) + 1/2 sum_i dx (n_i - n*_i)^2,
    differentiable in n0 (initial density, at rest, temperature T0), phi
    and sigma."""
    u0 = torch.zeros_like(n0)
    f0 = Equilibrium.apply(n0, u0, T0, solver)
    fN, flux = rollout(f0, phi, sigma, solver, nsteps, flux_node, every)
    nN = fN[0].sum(0)
    return dt * flux.sum() + 0.5 * dx * ((nN - target) ** 2).sum()
