"""Gradient of the flow's kinetic energy with respect to the body-force field.

Loss: E(F) = sum_x rho |u|^2 / 2 after ``nsteps`` steps from a fixed initial
state (the populations do not depend on F), with u from
Eq. velocitycalculation (so E depends on F also through the F/2 term).

Backward pass (discrete adjoint, project addition): the forward run keeps a
device copy of the state every K steps. For each segment, last to first, the
K-1 steps after its checkpoint are recomputed into a stash of K-1 buffers
(the checkpoint itself is the segment's first state), then K adjoint steps
run in reverse. With K >= nsteps the forward run writes every
state into a buffer of its own (nsteps population buffers, e.g. 113 GB for
500 steps at 128^3 in FP32) and the backward pass runs the adjoint steps only,
without recomputation; the gradient is bitwise the same. Every step's work is done by the library's
HIP kernels, a segment's steps in one call each (``cmlbm_steps_between``, ``cmlbm_steps_record``,
``cmlbm_adjoint_steps``: a call per step cost the host more than a step of a small box takes), with
``cmlbm_energy_seed`` and ``cmlbm_reduce``; torch provides buffers and copies.
"""
from __future__ import annotations

import torch

from .lattice import Lattice


def _on_stream_of(lat: Lattice, caller, work, *inputs: torch.Tensor):
    """work() with torch's part of it on the lattice's stream, where its kernels run: after
    what the caller queued so far, and before what the caller queues next. caller: the
    caller's current stream, or None where it is the lattice's; work returns
    (something for the caller to use, or None; the rest); inputs: the caller's
    tensors that it reads."""
    if caller is None:
        return work()
    lat.stream.wait_stream(caller)
    lat._after_use(*[t for t in inputs if t.device == lat.device])
    with torch.cuda.stream(lat.stream):
        out = work()
        if out[0] is not None:
            out[0].record_stream(caller)
    caller.wait_stream(lat.stream)
    return out


def _keep_all(nsteps: int, K: int) -> bool:
    return nsteps >= 1 and K >= nsteps


def _forward(lat: Lattice, F: torch.Tensor, f0_state: torch.Tensor, nsteps: int, K: int):
    """Run the forward pass from f0_state with force field F. Returns E, the
    checkpoints and a buffer of its own holding the final state fbar(nsteps),
    so that the backward pass does not depend on what the lattice does in
    between."""
    if nsteps < 0 or K < 1:
        raise ValueError(f"nsteps must be >= 0 and K >= 1 (got nsteps={nsteps}, K={K})")
    lat.set_force((0.0, 0.0, 0.0), F)
    cur = lat.state_buffer()
    if _keep_all(nsteps, K):
        # every state kept, ckpts[n] = fbar(n) for n < nsteps, in one allocation
        # whose last entry receives the last step and then holds fbar(nsteps)
        states = torch.empty((nsteps + 1,) + tuple(cur.shape), dtype=cur.dtype, device=cur.device)
        states[0].copy_(f0_state)
        lat.steps_record(states[0], states[1:])
        cur.copy_(states[nsteps])   # the lattice's state is fbar(nsteps) afterwards, as with checkpoints
        return lat.reduce()["ke"], states[:nsteps], states[nsteps]
    # the checkpoints, and the final state after them, in one allocation (one
    # request to the allocator instead of one per checkpoint)
    nseg = (nsteps + K - 1) // K
    states = torch.empty((nseg + 1,) + tuple(cur.shape), dtype=cur.dtype, device=cur.device)
    if lat.in_place or lat.sgs_force:
        # one buffer, or the sub-grid stress of the step before: the lattice's own
        # steps, a copy of its state after each segment (E only: no adjoint)
        cur.copy_(f0_state)
        for s in range(nseg):
            states[s].copy_(lat.state_buffer())
            lat.step(min(K, nsteps - s * K))
        states[nseg].copy_(lat.state_buffer())
    else:
        # the last step of each segment writes the next checkpoint, the first step
        # of each reads it: no copies of states but of the first and the last
        states[0].copy_(f0_state)
        for s in range(nseg):
            lat.steps_between(states[s], states[s + 1], min(K, nsteps - s * K))
        cur.copy_(states[nseg])
    return lat.reduce()["ke"], states[:nseg], states[nseg]


def _backward(lat: Lattice, F: torch.Tensor, ckpts, final: torch.Tensor, nsteps: int, K: int):
    """dE/dF for the forward pass that used force field F and left `final`.
    Binds F to the lattice again (the adjoint and the recomputed steps read
    it), so that other work on the lattice between the passes does not change
    the result; the lattice's state is not touched."""
    lat.set_force((0.0, 0.0, 0.0), F)
    lam = lat.lam_buffer()
    lam2 = torch.empty_like(lam)
    gF = torch.empty((3, lat.nz, lat.ny, lat.nx), dtype=lat.dtype, device=lat.device)
    lat.energy_seed(final, lam, gF)
    if nsteps == 0:   # E of the initial state: F enters only through u's F/2 term
        return gF
    if _keep_all(nsteps, K):
        lat.adjoint_steps(ckpts[0], ckpts[1:], lam, lam2, gF)
        return gF
    # the states of a segment after its checkpoint, which is only read and needs no
    # copy (one allocation: the first backward pass measured 1 % faster than with
    # K - 1 separate ones at 128^3, K = 50)
    block = torch.empty((K - 1,) + tuple(ckpts[0].shape), dtype=ckpts[0].dtype, device=ckpts[0].device)
    for s in range(len(ckpts) - 1, -1, -1):
        rest = block[:min(K, nsteps - s * K) - 1]
        lat.steps_record(ckpts[s], rest)
        lam, lam2 = lat.adjoint_steps(ckpts[s], rest, lam, lam2, gF)
    return gF


class EnergyAdjoint(torch.autograd.Function):
    """E = EnergyAdjoint.apply(F, lattice, f0_state, nsteps, K).

    F: (3, nz, ny, nx) force field in the lattice's compute dtype; f0_state: an
    internal-layout population buffer (e.g. a copy of ``lattice.state_buffer()``
    after ``init_equilibrium``). Returns E as a 0-d float64 tensor on the
    lattice's device; ``backward`` returns dE/dF. The forward pass keeps its own
    copies of F, of the checkpoints and of the final state, so several applies
    on one lattice, and steps or force changes between forward and backward,
    leave each gradient that of its own forward pass. After either pass the
    lattice's force field is the F of that pass. A lattice on a stream of its own
    works there; the caller's stream waits for it.
    """

    @staticmethod
    def forward(ctx, F, lat, f0_state, nsteps, K):
        def work():
            Fs = F.detach().to(device=lat.device, dtype=lat.dtype).clone()
            return (None, Fs) + _forward(lat, Fs, f0_state, int(nsteps), int(K))

        caller = torch.cuda.current_stream(lat.device.index)
        ctx.caller = None if caller == lat.stream else caller
        _, Fs, E, ckpts, final = _on_stream_of(lat, ctx.caller, work, F, f0_state)
        ctx.lat, ctx.F, ctx.ckpts, ctx.final = lat, Fs, ckpts, final
        ctx.nsteps, ctx.K = int(nsteps), int(K)
        return torch.tensor(E, dtype=torch.float64, device=F.device)

    @staticmethod
    def backward(ctx, gE):
        # (autograd makes the forward pass's stream the current one)
        gF, = _on_stream_of(ctx.lat, ctx.caller,
                            lambda: (_backward(ctx.lat, ctx.F, ctx.ckpts, ctx.final, ctx.nsteps, ctx.K),))
        ctx.ckpts = ctx.final = None
        return (gE.to(gF.dtype) * gF), None, None, None, None


def energy_and_grad(lat: Lattice, F: torch.Tensor, f0_state: torch.Tensor, nsteps: int, K: int = 50):
    """Convenience wrapper: (E, dE/dF)."""
    Fp = F.detach().clone().requires_grad_(True)
    E = EnergyAdjoint.apply(Fp, lat, f0_state, nsteps, K)
    E.backward()
    return float(E.detach()), Fp.grad
