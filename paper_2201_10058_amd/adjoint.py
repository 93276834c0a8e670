"""Gradients of final states with respect to initial positions, velocities and
masses, through trajectories of base steps (Appendix A of GENGA II, without
the direct solver), by the hand-written VJPs of libgenga.so.

The forward pass keeps a checkpoint of (x, v) every `checkpoint_every` steps.
The backward pass recomputes each segment from its checkpoint with the same
kernels (every kernel is deterministic; xa and xc are the positions the
operators' own calls give, which differ from the fused step's by rounding),
keeps the per-step intermediate states and applies the adjoints of the
operators in reverse order:

    rc = Rcrit(x0, v0, m)            -> rcrit_vjp
    v1 = v0 + h a(x0, m, rc)         -> kick_vjp(scale = h)
    xa = x0 + h P(v1, m) / m_star     -> hc_vjp
    (xb, v2) = Kepler(xa, v1; dt)    -> drift_vjp
    xc = xb + h P(v2, m) / m_star     -> hc_vjp
    v3 = v2 + h a(xc, m, rc)         -> kick_vjp(scale = h)
"""
from __future__ import annotations

import torch

from . import native as N

_XYZ = ("x", "y", "z")
_V = ("vx", "vy", "vz")


def _state(X, V, m, rc) -> N.State:
    return N.State({"x": X[0], "y": X[1], "z": X[2], "vx": V[0], "vy": V[1], "vz": V[2],
                    "m": m, "rc": rc})


class _Fixed(N.Config):
    """A pass's own configuration, never changed: its structure is filled once
    (several microseconds each time, at fourteen calls per step)."""

    def __init__(self, **values):
        super().__init__(**values)
        self._params = super().params()

    def params(self) -> N.Params:
        return self._params


class _Runner:
    def __init__(self, n, cfg: N.Config, device):
        if cfg.c_light or cfg.slevels > 1 or cfg.direct or cfg.tp_mode:
            # the adjoint covers the base step's operators only
            raise N.GengaError(N.E_UNSUPPORTED, "adjoint of a step with GR, levels, the direct "
                               "solver or test particles")
        flags, precision = N.FLAG_NOSYNC, cfg.precision
        if precision == N.MIXED and n < N.MIXED_STEP_MIN:
            # genga_step takes the binary64 kick here unless the caller sets the
            # kick's form or shape; every operator of the pass takes the same
            if cfg.ipt or cfg.slices or cfg.flags & (N.FLAG_DIRECTED | N.FLAG_SYMMETRIC):
                flags |= N.FLAG_DIRECTED
            else:
                precision = N.FP64
        self.cfg = _Fixed(**{**cfg.__dict__, "flags": flags, "precision": precision,
                             "events": (None,) * 4})
        self.ws = N.Workspace(n, self.cfg, device=device)
        self.h = 0.5 * cfg.dt

    def step(self, st):
        code = N.step(st, self.cfg, self.ws)
        if code not in (N.OK,):
            raise N.GengaError(code, "genga_step")

    def segment_saving(self, X, V, m, steps):
        """The steps of a segment from (X, V); per step the states that the
        adjoint needs: the step's input, that of the drift (after the first
        kick and HC) and its output after the second HC, with the step's
        radii.  The operators work in place, each on its own copy in one
        buffer.  The last step's second kick is left out: nothing reads it."""
        n, cfg, ws, h = m.shape[0], self.cfg, self.ws, self.h
        buf = torch.empty((3 * steps, 6, n), dtype=torch.float64, device=m.device)
        buf[0, :3].copy_(X)
        buf[0, 3:].copy_(V)
        S = buf.unbind(0)
        rows = buf.view(18 * steps, n).unbind(0)
        RC = torch.empty((steps, n), dtype=torch.float64, device=m.device).unbind(0)
        _state(buf[0, :3], buf[0, 3:], m, RC[0])    # checks m, as saved by the graph
        saved = []
        for k in range(steps):
            at = [rows[6 * (3 * k + j):6 * (3 * k + j + 1)] for j in range(3)]
            first, drift, second = st = [N.State._of_rows(r, m, RC[k]) for r in at]
            if k:
                # the second half kick of the step before, with its radii
                S[3 * k].copy_(S[3 * k - 1])
                N.kick(N.State._of_rows(at[0], m, RC[k - 1]), cfg, ws, h)
            N.rcrit(first, cfg, ws)
            S[3 * k + 1].copy_(S[3 * k])
            N.kick(drift, cfg, ws, h)
            N.hc(drift, cfg, ws, h)
            S[3 * k + 2].copy_(S[3 * k + 1])
            N.drift(second, cfg, ws, cfg.dt)
            N.hc(second, cfg, ws, h)
            saved.append(st)
        return saved

    def step_adjoint(self, saved, adj: N.AdjointState):
        """Reverse one step: adj holds (xbar, vbar) of the step's output on entry
        and of its input on exit; adj.m accumulates.  A kick's adjoint leaves
        vbar as it is, so the accelerations' adjoint is read there."""
        cfg, ws, h = self.cfg, self.ws, self.h
        first, drift, second = saved
        vbar = [adj.t[k] for k in _V]
        adj.t["rc"].zero_()
        # second half kick at (xc, m, rc): abar = h vbar
        N.kick_vjp(second, cfg, ws, h, vbar, adj)
        # HC at v2
        N.hc_vjp(second, cfg, ws, h, adj)
        # drift at its input (xa, v1)
        N.drift_vjp(drift, cfg, ws, cfg.dt, adj)
        # HC at v1
        N.hc_vjp(drift, cfg, ws, h, adj)
        # first half kick and critical radii at the step's input
        N.kick_vjp(first, cfg, ws, h, vbar, adj)
        N.rcrit_vjp(first, cfg, ws, adj)


class Trajectory(torch.autograd.Function):
    """(X0, V0, m) -> (X_T, V_T) after `steps` base steps.  X, V: (3, N)."""

    @staticmethod
    def forward(ctx, X0, V0, m, steps: int, cfg: N.Config, checkpoint_every: int = 20):
        device = X0.device
        n = X0.shape[1]
        run = _Runner(n, cfg, device)
        X = X0.detach().clone().contiguous()
        V = V0.detach().clone().contiguous()
        mm = m.detach().contiguous()
        rc = torch.zeros(n, dtype=torch.float64, device=device)
        ckpts = []
        st = _state(X, V, mm, rc)
        for k in range(steps):
            if k % checkpoint_every == 0:
                ckpts.append((k, X.clone(), V.clone()))
            run.step(st)
        code = N.read_status(run.ws)
        if code != N.OK:
            raise N.GengaError(code, "trajectory forward")
        ctx.save_for_backward(mm)
        ctx.ckpts = ckpts
        ctx.steps = steps
        ctx.cfg = cfg
        ctx.ce = checkpoint_every
        return X, V

    @staticmethod
    def backward(ctx, gX, gV):
        (m,) = ctx.saved_tensors
        n = m.shape[0]
        device = m.device
        run = _Runner(n, ctx.cfg, device)
        adj = N.AdjointState(n, device)
        gX = torch.zeros((3, n), dtype=torch.float64, device=device) if gX is None else gX
        gV = torch.zeros((3, n), dtype=torch.float64, device=device) if gV is None else gV
        for c, k in enumerate(_XYZ):
            adj.t[k].copy_(gX[c])
        for c, k in enumerate(_V):
            adj.t[k].copy_(gV[c])
        for (k0, Xc, Vc) in reversed(ctx.ckpts):
            k1 = min(k0 + ctx.ce, ctx.steps)
            for saved in reversed(run.segment_saving(Xc, Vc, m, k1 - k0)):
                run.step_adjoint(saved, adj)
        code = N.read_status(run.ws)
        if code != N.OK:
            raise N.GengaError(code, "trajectory backward")
        gX0 = torch.stack([adj.t[k] for k in _XYZ])
        gV0 = torch.stack([adj.t[k] for k in _V])
        return gX0, gV0, adj.t["m"].clone(), None, None, None


def simulate(X0, V0, m, steps: int, cfg: N.Config, checkpoint_every: int = 20):
    """Differentiable trajectory: returns (X_T, V_T); gradients flow to X0, V0, m."""
    return Trajectory.apply(X0, V0, m, steps, cfg, checkpoint_every)
