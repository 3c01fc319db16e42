"""Differentiable rollouts of the ESELBM step (torch.autograd front end).

Every step, loss and adjoint is a kernel of libeselbm.so; this module only
schedules them:

* ``Rollout.forward`` runs n steps, keeping the state every ``ckpt_every``
  steps (checkpoints) and, optionally, accumulating a dissipation loss
  weight * sum_x |omega|^2 after every step.  The step itself writes the
  velocity and density of its output (the loss depends on the state only
  through them), so the loss reads that field instead of the state.
  The states of the last ``keep_segments`` segments (those after the first
  kept segment's checkpoint; by default the last segment's only) are written
  to buffers of their own and kept, with their velocity fields, as is the
  velocity field of every checkpoint: the backward sweep starts from them.
  ``keep_segments=None`` keeps every state, so that the backward recomputes
  nothing (at 128^3 D3Q27 in single precision, 500 states take 113 GB of
  the 288 GB of HBM); ``keep_segments='auto'`` keeps as many trailing
  segments as fit a memory budget (by default 80% of the free device
  memory when the forward starts).
* ``Rollout.backward`` sweeps the checkpoint segments in reverse.  For each
  segment whose states were not kept it recomputes them from its checkpoint
  (with their velocity fields).  It then applies the adjoint step kernel from the
  segment's last state down to the first.  Each state's loss seed
  (dL/df_i = s0 + c_i.s) is added by the adjoint step that reads it; in
  single precision that step forms the seed itself from the state's
  velocity field, otherwise a seed pass writes it in compact form first.
  The adjoint kernel also accumulates the body-force gradient.

``GraphedRollout`` captures a rollout's forward and backward sweeps in two
HIP graphs for grids small enough that launches dominate.

Autograd functions wrap the three pieces of a training objective:
``equilibrium`` (initial state from rho, u; gradient w.r.t. u), ``rollout``
(state after n steps and the accumulated dissipation; gradients w.r.t. the
initial state and the force) and ``kinetic_energy`` (sum rho |u|^2 / 2).
"""
from __future__ import annotations

import torch

from .eselbm import Solver

# the calls that the solver's native sequences make in place of these methods
_SEQUENCE_CALLS = {
    "step_series": {m: getattr(Solver, m) for m in ("step", "set_velocity_field", "dissipation_loss_uv")},
    "adjoint_series": {m: getattr(Solver, m) for m in ("adjoint_step", "adjoint_step_diss")},
}


def _native(solver, series: str) -> bool:
    """Whether the solver has the native sequence and the methods it stands
    for are Solver's own, not a subclass's or an instance's."""
    return hasattr(solver, series) and all(
        getattr(getattr(solver, m), "__func__", None) is f for m, f in _SEQUENCE_CALLS[series].items())


class Rollout:
    def __init__(self, solver: Solver, tau: float, nsteps: int, ckpt_every: int,
                 diss_weight: float | None = None, keep_segments: int | str | None = 1,
                 memory_budget: float | None = None):
        if nsteps < 1 or ckpt_every < 1:
            raise ValueError("nsteps and ckpt_every must be >= 1")
        if keep_segments == "auto":
            pass
        elif keep_segments is not None and (isinstance(keep_segments, str) or int(keep_segments) < 1):
            raise ValueError("keep_segments must be >= 1, None or 'auto'")
        self.s = solver
        self.tau = float(tau)
        self.nsteps = int(nsteps)
        self.K = int(ckpt_every)
        self.diss_weight = diss_weight
        self.keep_segments = keep_segments if keep_segments in (None, "auto") else int(keep_segments)
        self.memory_budget = memory_budget
        self.kept = self.keep_segments if self.keep_segments != "auto" else 1
        self.ckpts: dict[int, torch.Tensor] = {}
        # velocity fields of the checkpoints (with the loss), and the states
        # of the last segment after its checkpoint with their velocity fields
        self.ckpt_uv: dict[int, torch.Tensor] = {}
        self.tail: dict[int, tuple[torch.Tensor, torch.Tensor | None]] = {}
        self.uv_end: torch.Tensor | None = None
        # whether _steps makes native calls (looked up at the start of a sweep)
        self.native = False

    def _steps(self, f: torch.Tensor, outs: list, uvs: list | None = None, loss: torch.Tensor | None = None):
        """One step f -> outs[0] -> outs[1] ... each; with ``uvs`` the velocity
        field of each, with ``loss`` (and ``uvs``) its dissipation loss added.
        One native call where the solver has it: on a small lattice the
        Python call of a step takes longer than the step."""
        s = self.s
        if not outs:
            return
        if self.native:
            s.step_series(f, outs, self.tau, uvs, loss if uvs is not None else None, self.diss_weight or 0.0)
            return
        for k, out in enumerate(outs):
            if uvs is None:
                s.step(f, out, 1, self.tau)
            else:
                s.set_velocity_field(uvs[k])
                try:
                    s.step(f, out, 1, self.tau)
                finally:
                    s.set_velocity_field(None)
                if loss is not None:
                    s.dissipation_loss_uv(uvs[k], loss=loss, weight=self.diss_weight)
            f = out

    def _last_start(self) -> int:
        """First state of the last checkpoint segment."""
        return ((self.nsteps - 1) // self.K) * self.K

    def _resolve_kept(self) -> int | None:
        """The trailing segments the forward keeps: keep_segments, or with
        'auto' as many as fit the memory budget (bytes; by default 80% of the
        device memory free now, the caching allocator's unused reserve
        included), at least one; None when that is all of them."""
        if self.keep_segments != "auto":
            return self.keep_segments
        s = self.s
        per_state = s.Q * s.cells * torch.empty((), dtype=s.storage_dtype).element_size()
        if self.diss_weight is not None:
            per_state += (s.D + 1) * s.cells * 4
        budget = self.memory_budget
        if budget is None:
            free, _ = torch.cuda.mem_get_info(s.device)
            free += torch.cuda.memory_reserved(s.device) - torch.cuda.memory_allocated(s.device)
            budget = 0.8 * free
        nseg = (self.nsteps + self.K - 1) // self.K
        k = max(1, int(budget // (self.K * per_state)))
        return None if k >= nseg else k

    def _kept_start(self) -> int:
        """First state (a checkpoint) of the first segment whose states the
        forward keeps."""
        if self.kept is None:
            return 0
        return max(0, self._last_start() - (self.kept - 1) * self.K)

    def forward(self, f0: torch.Tensor, loss_acc: torch.Tensor | None = None) -> torch.Tensor:
        """State after nsteps; with a dissipation weight, adds the loss of
        every state f^1..f^n to ``loss_acc`` (a device float64 scalar)."""
        s = self.s
        self.native = _native(s, "step_series")
        self.ckpts, self.ckpt_uv, self.tail, self.uv_end = {}, {}, {}, None
        self.kept = self._resolve_kept()
        cur = f0.clone()
        nxt = s.empty_state()
        self.ckpts[0] = cur.clone()
        with_loss = self.diss_weight is not None and loss_acc is not None
        uv = s.empty_velocity() if with_loss else None
        first = self._kept_start()
        # steps are handed over a checkpoint segment at a time (up to ``stop``)
        start = 0
        while start < self.nsteps:
            stop = min(start + self.K, self.nsteps)
            # the states after the first kept segment's checkpoint, and the
            # final one, get buffers of their own (the former are kept for
            # the backward)
            outs, uvs, src = [], [], cur
            for m in range(start + 1, stop + 1):
                keep = first < m < self.nsteps
                fresh = m > first
                out = s.empty_state() if fresh else nxt
                if not fresh:
                    nxt = src
                outs.append(out)
                uvs.append((s.empty_velocity() if (keep or m == first) else uv) if with_loss else None)
                if keep and m % self.K != 0:
                    self.tail[m] = (out, uvs[-1])
                src = out
            self._steps(cur, outs, uvs if with_loss else None, loss_acc)
            cur = src
            if stop % self.K == 0 and stop < self.nsteps:
                # a kept state's buffer is never written again
                self.ckpts[stop] = cur if stop > first else cur.clone()
                if with_loss:
                    self.ckpt_uv[stop] = uvs[-1] if stop >= first else uvs[-1].clone()
            start = stop
        if with_loss:
            self.uv_end = uvs[-1]
        return cur

    def backward(self, lam_final: torch.Tensor | None, diss_grad: float = 0.0,
                 force_grad: torch.Tensor | None = None) -> torch.Tensor:
        """Adjoint of the initial state given dL/df^n (may be None = 0) and the
        gradient of the accumulated dissipation loss; accumulates dL/dF."""
        s = self.s
        self.native, native = _native(s, "step_series"), _native(s, "adjoint_series")
        lam = s.empty_adjoint()
        if lam_final is None:
            lam.zero_()
        else:
            lam.copy_(lam_final)
        other = s.empty_adjoint()
        w = None if self.diss_weight is None else self.diss_weight * float(diss_grad)
        # The loss seed of state f^n enters the adjoint step that reads
        # lambda^n (the next one down).  In single precision that step forms
        # it itself from f^n's velocity field (pend_uv); otherwise a seed
        # pass writes it in compact per-cell form (pend_seed) and the step
        # adds it.
        fused = bool(w) and s.compute_dtype == torch.float32
        seed = s.empty_seed() if w else None
        pend_seed = pend_uv = None

        def seed_of(f_state, uv):
            nonlocal pend_seed, pend_uv
            if fused and uv is not None:
                pend_uv = uv
            elif uv is not None:
                s.dissipation_loss_uv(uv, seed=seed, weight=w, force_grad=force_grad)
                pend_seed = seed
            else:
                s.dissipation_seed(f_state, seed, weight=w, force_grad=force_grad)
                pend_seed = seed

        n_end = self.nsteps
        if w:
            if self.uv_end is not None:
                seed_of(None, self.uv_end)
            else:
                seed_of(self._state_at_end(), None)
        for start in sorted(self.ckpts, reverse=True):
            stop = min(start + self.K, n_end)
            # states f^start .. f^(stop-1) and, with the loss, the velocity
            # field of each (None where only the state is at hand)
            states = [self.ckpts[start]]
            uvs = [self.ckpt_uv.get(start)]
            kept = all(m in self.tail for m in range(start + 1, stop))
            if kept:
                states += [self.tail[m][0] for m in range(start + 1, stop)]
                uvs += [self.tail[m][1] for m in range(start + 1, stop)]
            else:
                fresh = [s.empty_state() for _ in range(start + 1, stop)]
                fuv = [s.empty_velocity() for _ in fresh] if w else None
                self._steps(states[0], fresh, fuv)
                states += fresh
                uvs += fuv if w else [None] * len(fresh)
            if kept:
                # the kept states now live in this segment's list only, so
                # they are freed with it, segment by segment (a later
                # backward of the same forward recomputes them)
                for m in range(start + 1, stop):
                    del self.tail[m]
            # the seed of the state after each step: none, or formed in the
            # step from its velocity field, or (w without such a field, or in
            # double precision) by a pass of its own
            if native and pend_seed is None and (
                    not w or (fused and all(u is not None for u in uvs[1:]) and (start == 0 or uvs[0] is not None))):
                lam, other = s.adjoint_series(states[::-1], lam, other, self.tau,
                                              [pend_uv] + uvs[:0:-1] if w else None, w or 0.0, force_grad)
                pend_uv = uvs[0] if w and start >= 1 else None
            else:
                for n in range(stop - 1, start - 1, -1):
                    f_n = states[n - start]
                    if pend_uv is not None:
                        s.adjoint_step_diss(f_n, lam, pend_uv, w, other, self.tau, force_grad=force_grad)
                    else:
                        s.adjoint_step(f_n, lam, other, self.tau, force_grad=force_grad, seed_next=pend_seed)
                    lam, other = other, lam
                    pend_seed = pend_uv = None
                    if w and n >= 1:
                        seed_of(f_n, uvs[n - start])
            del states, uvs
            n_end = start
        return lam

    def _state_at_end(self) -> torch.Tensor:
        last = max(self.ckpts)
        cur = self.ckpts[last].clone()
        nxt = self.s.empty_state()
        for _ in range(last, self.nsteps):
            self.s.step(cur, nxt, 1, self.tau)
            cur, nxt = nxt, cur
        return cur


class GraphedRollout:
    """A rollout captured in two HIP graphs, for grids where the kernel
    launches rather than the kernels set the time (a small 2-D lattice steps
    in a few microseconds).

    The forward graph runs ``Rollout.forward`` from the static state ``f0``
    (copy an initial state into it before each replay) and leaves the final
    state in ``fN`` and, with a dissipation weight, the accumulated loss in
    ``loss``.  The backward graph runs ``Rollout.backward`` from the static
    adjoint ``lam_final`` with the loss gradient ``diss_grad`` fixed at
    capture, and leaves the adjoint of ``f0`` in ``lam0`` and, with
    ``with_force_grad``, the gradient with respect to the solver's
    registered force in ``force_grad``.  A backward replay uses the states of
    the last forward replay; ``keep_segments`` chooses, as in ``Rollout``,
    which of them the forward graph keeps rather than the backward graph
    recomputing them.

    A replay relaunches the captured kernels on the same buffers: its results
    equal an eager rollout's bit for bit.  The solver's settings at capture
    (mode, force, walls) are part of the graphs.  Construction runs the
    rollout once eagerly (the first allocations of the caching allocator and
    of the library's loss scratch, which a capture may not make) and then
    captures; the library's calls in a rollout launch kernels and device
    copies only (no memset, no allocation, no synchronisation).
    """

    def __init__(self, solver: Solver, f0: torch.Tensor, tau: float, nsteps: int, ckpt_every: int,
                 diss_weight: float | None = None, diss_grad: float = 1.0, with_force_grad: bool = False,
                 keep_segments: int | str | None = 1):
        s = solver
        self.ro = Rollout(s, tau, nsteps, ckpt_every, diss_weight, keep_segments)
        self.f0 = f0.detach().clone()
        self.lam_final = s.empty_adjoint().zero_()
        self.loss = torch.zeros(1, dtype=torch.float64, device=s.device)
        self.force_grad = (torch.zeros((s.D,) + s.shape, dtype=torch.float32, device=s.device)
                           if with_force_grad else None)
        with_loss = diss_weight is not None

        def fwd():
            self.loss.zero_()
            return self.ro.forward(self.f0, self.loss if with_loss else None)

        def bwd():
            if self.force_grad is not None:
                self.force_grad.zero_()
            return self.ro.backward(self.lam_final, diss_grad=diss_grad, force_grad=self.force_grad)

        cur = torch.cuda.current_stream(s.device)
        side = torch.cuda.Stream(device=s.device)
        side.wait_stream(cur)
        with torch.cuda.stream(side):
            fwd()
            bwd()
        cur.wait_stream(side)
        torch.cuda.synchronize(s.device)
        self._gf = torch.cuda.CUDAGraph()
        self._gb = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self._gf):
            self.fN = fwd()
        # every state the backward graph reads, held here whatever the
        # backward sweep does with its own references
        self._reads = (dict(self.ro.ckpts), dict(self.ro.ckpt_uv), dict(self.ro.tail), self.ro.uv_end)
        with torch.cuda.graph(self._gb):
            self.lam0 = bwd()

    def forward(self):
        """Replays the forward graph: (fN, loss)."""
        self._gf.replay()
        return self.fN, self.loss

    def backward(self):
        """Replays the backward graph: (lam0, force_grad)."""
        self._gb.replay()
        return self.lam0, self.force_grad


class _Equilibrium(torch.autograd.Function):
    @staticmethod
    def forward(ctx, rho, u, solver):
        ctx.solver = solver
        ctx.save_for_backward(rho, u)
        return solver.init_equilibrium(rho.contiguous(), u.contiguous())

    @staticmethod
    def backward(ctx, gf):
        rho, u = ctx.saved_tensors
        s = ctx.solver
        gu = s.equilibrium_vjp(rho, u, gf.to(s.compute_dtype).contiguous())
        return None, gu, None


class _Rollout(torch.autograd.Function):
    @staticmethod
    def forward(ctx, f0, force, solver, tau, nsteps, ckpt_every, diss_weight, keep_segments):
        # the rollout's force replaces whatever the solver had registered
        # (None clears it), so the forward never runs with a stale force that
        # the backward would not differentiate
        solver.set_force(None if force is None else force.detach().contiguous())
        ro = Rollout(solver, tau, nsteps, ckpt_every, diss_weight, keep_segments)
        loss = torch.zeros(1, dtype=torch.float64, device=f0.device)
        fN = ro.forward(f0.detach().contiguous(), loss if diss_weight is not None else None)
        ctx.ro = ro
        ctx.has_force = force is not None
        return fN, loss[0]

    @staticmethod
    def backward(ctx, g_fN, g_loss):
        ro = ctx.ro
        s = ro.s
        fg = None
        if ctx.has_force:
            fg = torch.zeros((s.D,) + s.shape, dtype=torch.float32, device=s.device)
        lamN = None if g_fN is None else g_fN.to(s.compute_dtype).contiguous()
        dl = 0.0 if g_loss is None else float(g_loss)
        lam0 = ro.backward(lamN, diss_grad=dl, force_grad=fg)
        return lam0, fg, None, None, None, None, None, None


class _Kinetic(torch.autograd.Function):
    @staticmethod
    def forward(ctx, f, solver):
        ctx.solver = solver
        ctx.save_for_backward(f)
        loss = torch.zeros(1, dtype=torch.float64, device=f.device)
        solver.kinetic_loss(f.detach().contiguous(), loss=loss)
        return loss[0]

    @staticmethod
    def backward(ctx, g):
        (f,) = ctx.saved_tensors
        s = ctx.solver
        lam = s.empty_adjoint()
        s.kinetic_loss(f.contiguous(), lam=lam, scale=float(g))
        return lam, None


def equilibrium(solver: Solver, rho: torch.Tensor, u: torch.Tensor) -> torch.Tensor:
    return _Equilibrium.apply(rho, u, solver)


def rollout(solver: Solver, f0: torch.Tensor, tau: float, nsteps: int, ckpt_every: int,
            force: torch.Tensor | None = None, diss_weight: float | None = None,
            keep_segments: int | str | None = 1):
    """(state after nsteps, accumulated dissipation loss).  ``force`` becomes
    the solver's registered body force for the rollout; None clears it.
    ``keep_segments``: the trailing checkpoint segments whose states the
    forward keeps for the backward (None: all of them, no recomputation;
    'auto': as many as fit 80% of the free device memory)."""
    return _Rollout.apply(f0, force, solver, tau, nsteps, ckpt_every, diss_weight, keep_segments)


def kinetic_energy(solver: Solver, f: torch.Tensor) -> torch.Tensor:
    return _Kinetic.apply(f, solver)
