"""Differentiable MPM rollouts through the hand-written adjoints, with substep
checkpointing.

The reconstruction of Sec. 3.3 optimises the wind force field F_w (and can
differentiate the material parameters theta) by gradient descent through the
simulation S of Eq. simulation_mpm.  `Rollout` runs n substeps of S on the
device with a force-grid wind (one field per time slot, piecewise constant
over the substeps) and exposes them to torch as one autograd Function.

Memory: the forward keeps the particle state every `ckpt` substeps only.  The
backward walks the segments in reverse; for each it re-runs the segment from
its checkpoint, keeping every substep's particle state, sort workspace and
grid (m, mv, v: about 28 B per grid node and 20 B per particle per substep),
then for every substep (last first) applies the adjoints in reverse order
(the last segment is kept by the forward and re-run only if another rollout
of the plan has used its store since): G2P adjoint (sorted scatter into the grid adjoint), grid-update adjoint with
the wind transpose into W_bar, P2G adjoint (per-particle gather, also giving
E_bar).  The substep loops run in the library (mpm_rollout, mpm_rollout_adj);
torch provides device memory and the final loss.

With `deterministic` every reduction of the forward and reverse substeps
runs in a fixed order (sort, P2G, the reverse G2P's grid scatter, the E and
force-grid adjoints), so a rollout's gradients are bit-identical run to run.

With `xref` the positions are xref + x: the rollout's x input and output are
displacements from that fixed reference (see the header), which keeps their
float32 resolution on the motion.

A particle whose stencil leaves the grid is skipped by the kernels and
flagged in the workspace status word (as are non-finite positions); the
status of every forward and recomputed substep is OR-ed on the device and
checked once per forward and once per backward, and a flagged rollout
raises instead of returning a truncated gradient.
"""
from __future__ import annotations

import torch

from . import api


class RolloutPlan:
    """Device buffers and constants for rollouts of one particle set on one grid."""

    def __init__(self, grid: dict, n: int, mass, vol0, region, nu, pin, dt: float, gravity, material: int,
                 bound: int, nw, box_lo, box_hi, K: int, n_sub: int, ckpt: int = 16, device="cuda",
                 xref=None, deterministic: bool = False):
        self.grid = api.make_grid(grid["nx"], grid["ny"], grid["nz"], grid["dx"], grid["origin"])
        self.N = grid["nx"] * grid["ny"] * grid["nz"]
        self.n = n
        self.mass, self.vol0, self.region, self.nu = mass, vol0, region, nu
        self.pin = pin
        self.xref = xref
        self.deterministic = bool(deterministic)
        self.prm = api.make_mpm_params(dt, gravity, bound, material, deterministic=self.deterministic)
        self.nw, self.box_lo, self.box_hi, self.K = tuple(nw), tuple(box_lo), tuple(box_hi), K
        self.n_sub, self.ckpt = n_sub, ckpt
        f = dict(dtype=torch.float32, device=device)
        self.device = device
        self.ws = api.alloc_workspace(self.grid, n, device, deterministic=self.deterministic)
        self._grids = torch.zeros(7, self.N, **f)
        self.gm, self.gmv, self.gv = self._grids[0], self._grids[1:4], self._grids[4:7]
        # grid adjoints in one buffer, cleared with one fill per substep_adjoint
        self._gbar = torch.zeros(10, self.N, **f)
        self.gvb, self.gmb, self.gmvb, self.accb = (self._gbar[0:3], self._gbar[3], self._gbar[4:7],
                                                    self._gbar[7:10])
        self._seg = None  # store of a segment's substeps, made when a gradient is first asked for
        self._seg_views = None  # segment_buffers' own
        self._kept = None  # token of the rollout whose last segment is in the store
        self._status = torch.zeros(1, dtype=torch.int32, device=device)  # OR of the substeps' status words

    def _segment_store(self):
        """Workspaces (ckpt, bytes), grids (ckpt, 7, N) and states between the
        substeps (ckpt - 1, 24 n) of a segment."""
        if self._seg is None:
            f = dict(dtype=torch.float32, device=self.device)
            nb = self.ws.numel()
            ws = torch.empty(self.ckpt * nb + 256, dtype=torch.uint8, device=self.device)
            off = (-ws.data_ptr()) % 256
            self._seg = (ws[off:off + self.ckpt * nb].view(self.ckpt, nb), torch.empty(self.ckpt, 7, self.N, **f),
                         torch.empty(max(self.ckpt - 1, 1), 24 * self.n, **f))
        return self._seg

    def segment_buffers(self):
        """Sort workspaces and grids (m, mv, v) for the substeps of one segment."""
        if self._seg_views is None:
            f = dict(dtype=torch.float32, device=self.device)
            self._seg_views = [(api.alloc_workspace(self.grid, self.n, self.device, deterministic=self.deterministic),
                                torch.empty(self.N, **f), torch.empty(3, self.N, **f), torch.empty(3, self.N, **f))
                               for _ in range(self.ckpt)]
        return self._seg_views

    def slot(self, s: int) -> int:
        return s * self.K // self.n_sub

    def particles(self, x, v, C, H, E):
        return api.ParticleArrays(x, v, C, H, self.mass, self.vol0, self.region, E, self.nu, self.xref)

    def check_status(self, what: str):
        """Raise if a substep since the last check met a particle outside the
        grid or a non-finite position (one host synchronisation)."""
        st = int(self._status.item())
        self._status.zero_()
        bad = st & (api.STATUS_OUT_OF_GRID | api.STATUS_NONFINITE)
        if bad:
            raise api.DiffWindError(f"rollout {what}: status {st:#x} (a particle left the grid or is not finite); "
                                    "the kernels skipped it, so the result would be truncated")

    def wind(self, W, s):
        return api.wind_force_grid(W[self.slot(s)], self.nw, self.box_lo, self.box_hi,
                                   deterministic=self.deterministic)

    def segment(self, W, s0: int, grids, ws, states=None) -> api.Segment:
        """The checkpoint segment that starts at substep s0; with states its
        substeps keep their own grids and workspaces."""
        count = min(self.ckpt, self.n_sub - s0)
        W[self.slot(s0 + count - 1)]  # an IndexError if W lacks a slot
        return api.rollout_segment(s0, count, self.n_sub, self.K, W.stride(0), grids, ws, states)

    # --------------------------------------------------------------- forward
    def substep(self, p: api.ParticleArrays, W, s: int, out=None, bufs=None, g2p: bool = True):
        """One substep; in place unless `out` = (x, v, C, H) buffers are given.
        `bufs` = (workspace, m, mv, v) keeps this substep's sort and grid."""
        ws, gm, gmv, gv = bufs if bufs is not None else (self.ws, self.gm, self.gmv, self.gv)
        api.mpm_sort(self.grid, self.prm, p.x, ws, xref=self.xref)
        api.mpm_p2g(self.grid, self.prm, p, gm, gmv, ws)
        self._status.bitwise_or_(ws[:4].view(torch.int32))
        api.mpm_grid_update(self.grid, self.prm, gm, gmv, self.wind(W, s), self.pin, gv, ws)
        if not g2p:
            return None
        if out is None:
            api.mpm_g2p(self.grid, self.prm, gv, p, p.x, p.v, p.C, p.F)
            return p
        api.mpm_g2p(self.grid, self.prm, gv, p, *out)
        return self.particles(*out, p.E)

    # -------------------------------------------------------------- backward
    def substep_adjoint(self, p: api.ParticleArrays, W, s: int, bar_out, bar_in, W_bar, E_bar, bufs=None):
        """Adjoint of substep s at input state p: adds into bar_in = (x, v, C, H)
        adjoints of the inputs, W_bar and E_bar, given bar_out of the outputs.
        `bufs` = the substep's kept (workspace, m, mv, v); without it the
        substep's grid is recomputed first."""
        g, prm = self.grid, self.prm
        wind = self.wind(W, s)
        if bufs is None:
            self.substep(p, W, s, g2p=False)
            bufs = (self.ws, self.gm, self.gmv, self.gv)
        ws, gm, gmv, gv = bufs
        self._gbar.zero_()
        xb, vb, Cb, Hb = bar_in
        api.mpm_g2p_adj(g, prm, gv, p, *bar_out, x_bar=xb, F_bar=Hb, grid_v_bar=self.gvb, ws=ws)
        api.mpm_grid_update_adj(g, prm, gm, gmv, wind, self.pin, self.gvb, self.gmb, self.gmvb, self.accb, ws)
        api.wind_to_grid_adj(g, wind, self.accb, W_bar[self.slot(s)])
        api.mpm_p2g_adj(g, prm, p, self.gmb, self.gmvb, xb, vb, Cb, Hb, E_bar, ws=ws)


class _RolloutFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, plan: RolloutPlan, keep: bool, W, E, x0, v0, C0, H0):
        W = W.detach().contiguous()
        E = E.detach().contiguous()
        state = [t.detach().clone() for t in (x0, v0, C0, H0)]
        ckpts = []
        for s0 in range(0, plan.n_sub, plan.ckpt):
            # a segment leaves its first state as it is: that is the checkpoint
            ckpts.append(state)
            out = [torch.empty_like(t) for t in state]
            if keep and s0 + plan.ckpt >= plan.n_sub:
                # the backward starts with this segment
                plan._kept = None
                ws, grids, states = plan._segment_store()
                seg = plan.segment(W, s0, grids, ws, states)
            else:
                seg = plan.segment(W, s0, plan._grids, plan.ws)
            api.mpm_rollout(plan.grid, plan.prm, plan.particles(*state, E), out, plan.wind(W, 0), plan.pin, seg,
                            plan._status)
            state = out
        plan.check_status("forward")
        ctx.kept = plan._kept = object() if keep and ckpts else None
        ctx.plan = plan
        ctx.ckpts = ckpts
        ctx.save_for_backward(W, E)
        return tuple(state)

    @staticmethod
    def backward(ctx, xb, vb, Cb, Hb):
        plan = ctx.plan
        W, E = ctx.saved_tensors
        W_bar = torch.zeros_like(W)
        E_bar = torch.zeros_like(E)
        ws, grids, states = plan._segment_store()
        kept = ctx.kept is not None and plan._kept is ctx.kept
        plan._kept = None
        # particle-state adjoints: two groups of packed (x, v, C, H)
        shapes = [t.shape for t in ctx.ckpts[0]]
        sizes = [t.numel() for t in ctx.ckpts[0]]
        pair = torch.empty(2, sum(sizes), dtype=torch.float32, device=W.device)
        groups = [list(t.view(sh) for t, sh in zip(torch.split(pair[k], sizes), shapes)) for k in range(2)]
        cur = 0
        for dst, b in zip(groups[cur], (xb, vb, Cb, Hb)):
            dst.zero_() if b is None else dst.copy_(b)
        plan.gvb.zero_()  # and zero again after each substep
        wind = plan.wind(W, 0)
        for k in reversed(range(len(ctx.ckpts))):
            # re-run the segment, keeping each substep's state, sort and grid
            seg = plan.segment(W, k * plan.ckpt, grids, ws, states)
            p = plan.particles(*ctx.ckpts[k], E)
            if not (kept and k == len(ctx.ckpts) - 1):
                api.mpm_rollout(plan.grid, plan.prm, p, None, wind, plan.pin, seg, plan._status)
            api.mpm_rollout_adj(plan.grid, plan.prm, p, wind, plan.pin, seg, pair, cur, plan._gbar, W_bar, E_bar)
            cur ^= seg.count & 1
        plan.check_status("backward")
        return (None, None, W_bar, E_bar, *[b.clone() for b in groups[cur]])


def rollout(plan: RolloutPlan, W, E, x0, v0, C0, H0):
    """Differentiable n-substep rollout: returns the final (x, v, C, H), with
    gradients flowing to W (K, 3, nw^3), E (n_regions,) and the initial state.
    With plan.xref set, x0 and the returned x are displacements from it.
    Raises DiffWindError if a particle left the grid."""
    args = (W, E, x0, v0, C0, H0)
    return _RolloutFn.apply(plan, torch.is_grad_enabled() and any(t.requires_grad for t in args), *args)
