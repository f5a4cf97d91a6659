"""Gradient of the mean flux (permeability) with respect to a per-cell
partial-bounce-back solid fraction, through the hand-written adjoint step.

Forward: T TRT sweeps from rest with solid fraction ns; J = mean over listed
cells of u_x = j_x + G_x/2 after the last sweep (permeability k = nu J / G_x).
Backward, two schedules over the same kernels (bitwise the same gradient):
  * two-level checkpointing -- the forward keeps the state every k steps;
    the backward walks the segments in reverse, recomputes the states of one
    segment into a buffer, and applies the adjoint step from the last state
    of the segment down to its first.  Memory: ceil(T/k) checkpoints + k
    buffer states; work: one extra forward sweep per step.
  * binomial ("revolve") checkpointing with a fixed number of snapshot slots
    (checkpointing.Revolve): memory snapshots + 3 states, work the optimal
    number of recomputed sweeps for that memory.
"""
from __future__ import annotations

import ctypes as C

import torch

from . import _native as N
from .checkpointing import Revolve
from .lattice import Compressed, Lattice, compress, init, narrow, objective


def _run_params(prm, n: int):
    """prm for the single sweeps of a longer run: without launch hints where a
    call of several sweeps over n cells would not follow them."""
    quiet = N.lbm_params.from_buffer_copy(prm)
    quiet.flags &= ~(N.FLAG_NONTEMPORAL | 0xff << N.FLAG_XCD_CHUNK_SHIFT)
    same = N.lbm_sweep_launch(prm, n, 2, 1) == N.lbm_sweep_launch(quiet, n, 2, 1)
    return quiet if same else prm


class _Steps:
    """Sweeps and adjoint steps over the first n cells of a list and its codes,
    on the stream that is current when this is made.  What does not change from call to call
    is resolved once: a small box is stepped as fast as its calls are issued."""

    def __init__(self, lat: Lattice, n: int, prm, comp: Compressed, ns: torch.Tensor | None):
        lib = N.load()
        run_prm = _run_params(prm, n)
        self.keep = (lat, prm, run_prm, comp, ns)
        lists = (n, lat.stride, comp.codes8.data_ptr(), comp.codes.data_ptr(),
                 comp.tile_records.data_ptr(), lat.adj.data_ptr())
        ns_ptr, stream = N._ptr(ns), N._stream()
        step, adjoint = lib.lbm_step_c8, lib.lbm_step_adjoint_c8
        head, adjoint_head = (C.byref(run_prm), *lists), (C.byref(prm), *lists)

        def sweeps(src: torch.Tensor, dst: torch.Tensor, k: int = 1):
            """k sweeps from src, alternating between dst and src (dst first)."""
            rc = step(*head, ns_ptr, src.data_ptr(), dst.data_ptr(), k, stream)
            if rc:
                N._check("lbm_step_c8", rc)

        def adjoint_step(f_t, lam_next, lam_t, grad):
            rc = adjoint(*adjoint_head, f_t.data_ptr(), ns_ptr, lam_next.data_ptr(),
                         lam_t.data_ptr(), grad.data_ptr(), stream)
            if rc:
                N._check("lbm_step_adjoint_c8", rc)

        self.sweeps, self.adjoint_step = sweeps, adjoint_step

    def advance(self, src, a, b, k: int):
        """State k sweeps after src, src itself left as it is: the first sweep
        reads it, the others alternate between a and b.  Returns (the array
        that holds the result, the other one); b may be None if k is 1."""
        self.sweeps(src, a)
        if k == 1:
            return a, b
        self.sweeps(a, b, k - 1)
        return (b, a) if (k - 1) % 2 else (a, b)


def codes_of(lat: Lattice, comp: Compressed | None) -> Compressed:
    """The lattice's 16-bit codes with their 8-bit form (built if not given)."""
    comp = compress(lat) if comp is None else comp
    return narrow(comp) if comp.codes8 is None else comp


def forward_states(lat: Lattice, prm, ns: torch.Tensor, T: int, k: int,
                   comp: Compressed | None = None):
    """Run T steps from rest; return (J, checkpoints at 0, k, 2k, ..., final state).

    The sweeps read the 8-bit adjacency codes where a tile allows them and
    the 16-bit codes elsewhere (bitwise the same states as the sweep over the
    full list, fewer bytes)."""
    comp = codes_of(lat, comp)
    assert comp.n == lat.base + lat.n_fluid and comp.codes.shape[1] == lat.stride
    st = init(lat, prm, ns=ns)
    steps = _Steps(lat, st.n, st.first_params, comp, ns)
    ckpts = []
    cur, spare = st.f, st.g
    t = 0
    while t < T:
        n = min(k, T - t)
        if T <= k:
            # one checkpoint: copied, since the state's two arrays are one
            # allocation, which a checkpoint in it would hold whole
            ckpts.append(cur.clone())
            steps.sweeps(cur, spare, n)
            if n % 2:
                cur, spare = spare, cur
        else:
            # the array that holds the state is the checkpoint (nothing writes
            # it again); the segment goes on in two others and ends in the
            # first of them, so the second checkpoint is the second of the
            # state's own two arrays
            ckpts.append(cur)
            out = torch.empty_like(cur) if spare is None else spare
            spare = torch.empty_like(cur) if n > 1 else None
            steps.advance(cur, *((out, spare) if n % 2 else (spare, out)), n)
            cur = out
        t += n
    st.f, st.g = cur, torch.empty_like(cur) if spare is None else spare
    st.steps += T
    J = objective(st)[0]  # mean x velocity, formed in the library (lbm_objective)
    return J, ckpts, st


def _as_state(ckpt: torch.Tensor, like: torch.Tensor) -> torch.Tensor:
    """A caller's checkpoint as the kernels read it: itself, or a copy laid out
    like `like` if it is kept elsewhere or in another form."""
    if (ckpt.shape == like.shape and ckpt.dtype == like.dtype and ckpt.device == like.device
            and ckpt.is_contiguous()):
        return ckpt
    return torch.empty_like(like).copy_(ckpt)


def adjoint_gradient(lat: Lattice, prm, ns: torch.Tensor, T: int, k: int, ckpts=None,
                     comp: Compressed | None = None):
    """dJ/dns [stride] (float64) by checkpointed reverse sweeps (the segment
    recomputation and the adjoint steps read the 8-bit codes in narrow tiles
    and the 16-bit codes elsewhere, as the forward does)."""
    comp = codes_of(lat, comp)
    if ckpts is None:
        _, ckpts, _ = forward_states(lat, prm, ns, T, k, comp)
    S, n = lat.stride, lat.n_fluid
    dev = lat.device
    lam = torch.empty((19, S), dtype=torch.float64, device=dev)
    lam_prev = torch.empty_like(lam)
    grad = torch.zeros(S, dtype=torch.float64, device=dev)
    N._check("lbm_step_adjoint", N.lbm_step_adjoint(prm, n, S, lat.adj, None, ns, None, lam, None))
    steps = _Steps(lat, n, prm, comp, ns)
    # states of a segment after its first, which is the checkpoint itself
    buf = [torch.empty_like(lam) for _ in range(min(k, T) - 1)] if ckpts else []
    # checkpoints at T and later (of a longer run) are not needed
    for s in reversed(range(min(len(ckpts), -(-T // k)))):
        t0 = s * k
        n_seg = min(t0 + k, T) - t0
        states = [_as_state(ckpts[s], lam)] + buf[:n_seg - 1]
        for j in range(1, n_seg):
            steps.sweeps(states[j - 1], states[j])
        for f_t in reversed(states):
            steps.adjoint_step(f_t, lam, lam_prev, grad)
            lam, lam_prev = lam_prev, lam
    return grad


def adjoint_gradient_revolve(lat: Lattice, prm, ns: torch.Tensor, T: int, snapshots: int,
                             comp: Compressed | None = None, stats: dict | None = None):
    """dJ/dns [stride] (float64) with binomial checkpointing: the reverse
    sweep starts from the initial state alone and keeps at most `snapshots`
    intermediate states (plus the initial one, a work state and the sweep's
    second array); the states are recomputed by the schedule of
    checkpointing.Revolve.  Bitwise the two-level gradient.  stats, if
    given, receives the forward sweeps the schedule ran."""
    comp = codes_of(lat, comp)
    S, n = lat.stride, lat.n_fluid
    dev = lat.device
    st0 = init(lat, prm, ns=ns)
    plan = Revolve(T, snapshots)
    slots = [st0.f] + [torch.empty_like(st0.f) for _ in range(snapshots + 1)]
    spare = st0.g  # the sweep's second array
    lam = torch.empty((19, S), dtype=torch.float64, device=dev)
    lam_prev = torch.empty_like(lam)
    grad = torch.zeros(S, dtype=torch.float64, device=dev)
    N._check("lbm_step_adjoint", N.lbm_step_adjoint(prm, n, S, lat.adj, None, ns, None, lam, None))
    lams = [lam, lam_prev]
    swept = [0]
    steps = _Steps(lat, n, prm, comp, ns)

    def advance(src, dst, t, k):
        # no copy: the sweeps after the first alternate between slot dst and
        # the spare array so that the last one writes slot dst
        a, b = (slots[dst], spare) if (k - 1) % 2 == 0 else (spare, slots[dst])
        steps.advance(slots[src], a, b, k)
        swept[0] += k

    def adjoint(slot, t):
        steps.adjoint_step(slots[slot], lams[0], lams[1], grad)
        lams.reverse()

    plan.run(advance, adjoint)
    assert swept[0] == plan.forward_steps
    if stats is not None:
        stats["forward_sweeps"] = swept[0]
        stats["states_held"] = snapshots + 3
    return grad


class PermeabilityFn(torch.autograd.Function):
    """J = PermeabilityFn.apply(ns, lattice, params, T, k[, snapshots]): mean x
    velocity after T sweeps; backward returns dJ/dns via the adjoint, with
    two-level checkpoints every k steps, or, if snapshots is given, with
    binomial checkpointing in that many snapshot slots (k unused)."""

    @staticmethod
    def forward(ctx, ns, lat, prm, T, k, *snapshots_arg):
        if prm.storage not in (N.STORAGES["f64"], N.STORAGES["f64s"]):
            raise ValueError("the adjoint needs FP64 storage")
        snapshots = snapshots_arg[0] if snapshots_arg else None
        ctx.n_inputs = 5 + len(snapshots_arg)
        nsd = ns.detach().contiguous()
        comp = codes_of(lat, None)
        if snapshots is None:
            J, ckpts, _ = forward_states(lat, prm, nsd, T, k, comp)
        else:
            J, ckpts = forward_states(lat, prm, nsd, T, max(T, 1), comp)[0], None
        ctx.lat, ctx.prm, ctx.T, ctx.k, ctx.snapshots = lat, prm, T, k, snapshots
        ctx.ckpts, ctx.comp = ckpts, comp
        ctx.save_for_backward(nsd)
        return J

    @staticmethod
    def backward(ctx, gJ):
        (ns,) = ctx.saved_tensors
        if ctx.snapshots is None:
            grad = adjoint_gradient(ctx.lat, ctx.prm, ns, ctx.T, ctx.k, ctx.ckpts, ctx.comp)
        else:
            grad = adjoint_gradient_revolve(ctx.lat, ctx.prm, ns, ctx.T, ctx.snapshots, ctx.comp)
        ctx.ckpts = ctx.comp = None
        return (grad * gJ,) + (None,) * (ctx.n_inputs - 1)
