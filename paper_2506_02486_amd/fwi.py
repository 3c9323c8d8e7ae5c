"""FWI gradient with respect to squared slowness m = 1/v^2 (adjoint-state method).

The forward model is the leapfrog step of the library (Dirichlet halos, optional
sponge), a Ricker source and receivers; the misfit is any function of the synthetic
traces.  ``FWIGrad.apply(m, problem)`` returns the traces and, on ``backward``, the
gradient of the loss with respect to m, computed by

* a forward sweep that keeps ``(u^{n-1}, u^n)`` every ``checkpoint_every`` steps
  (one native step loop, fd_forward_run, per checkpoint interval),
* a reverse sweep over the segments, last first: each segment is recomputed from its
  checkpoint, keeping s_n = L u^n + f^n of every step (fd_forward_keep), then for n
  descending the adjoint step forms the adjoint field at n from those at n+1 and n+2,
  with the gradient terms of the kept s_n and the trace residual of step n-1 added in
  its launch (fd_adjoint_run),
* the final scaling of the accumulated gradient to grad_m.

The adjoint runs by default in the scaled variable b = vdt2 D lambda
(``fd_adjoint_step_scaled``, ``fd_scatter_add_scaled``, ``fd_grad_finalize_scaled``):
there it is the forward update run backward in time, on the forward kernel, and
g_b = sum b^{n+1} (L u^n + f^n) gives grad_m = -g_b vdt2 / dt^2.  ``scaled=False``
runs it in lambda (``fd_adjoint_step``: lambda^n = 2 D lambda^{n+1} +
L(vdt2 D lambda^{n+1}) - E D lambda^{n+2}, g += D lambda^{n+1} (L u^n + f^n),
``fd_scatter_add``, ``fd_grad_finalize``: grad_m = -g vdt2^2 / dt^2).

Volumes held at once beside m and vdt2: with checkpoints every C steps, S segments, 2 (S - 1)
checkpoints, C kept sums, three wavefields and three of the adjoint; with C = 0 nt kept sums
and three more (unscaled four).

dt and the sponge are fixed when the problem is built (they do not depend on m).
All device work runs in libfd's kernels; torch allocates buffers and copies
checkpoints.
"""
from __future__ import annotations

import numpy as np
import torch

from . import api

# checkpoint intervals up to which the scaled reverse sweep takes a segment's last step on
# the wavefield itself (see _backward_scaled)
DIRECT_STEPS = 4


class FWIProblem:
    """One shot of an FWI gradient: geometry, time axis, source, receivers."""

    def __init__(self, shape, dt: float, src, rec: np.ndarray, nt: int, d=(10.0, 10.0, 10.0),
                 sponge_width: int = 16, sponge_vmax: float | None = None,
                 f0: float = api.RICKER_F0, t0: float | None = None,
                 checkpoint_every: int = 32, device="cuda"):
        nx, ny, nz = shape
        self.grid = g = api.Grid(nx, ny, nz, d)
        self.dt = float(dt)
        self.nt = int(nt)
        self.src = tuple(int(x) for x in src)
        self.device = device
        # checkpoint_every = 0 keeps s_n = L u^n + f^n of every step (nt volumes: 89 GB
        # at 256^3 and 1000 steps fits one MI355X's 288 GB) and skips the recompute
        self.C = int(checkpoint_every)
        if self.C < 0:
            raise ValueError("checkpoint_every must be >= 0 (0: keep every state)")
        if sponge_width > 0:
            if sponge_vmax is None:
                raise ValueError("a sponge needs the (fixed) vmax it is designed for")
            self.sponge = api.Sponge(g, sponge_width, sponge_vmax, self.dt, device=device)
        else:
            self.sponge = None
        self.w = api.ricker(self.nt, self.dt, f0, t0)
        self.rec_off = torch.from_numpy(g.offsets(rec)).to(device)
        self.rec_plane = api.receiver_plane(g, rec, device)  # sampled in the stencil launch
        self.nrec = self.rec_off.numel()
        self.src_off = torch.from_numpy(g.offsets(np.array([self.src], np.int32))).to(device)
        self.m = g.zeros(device)
        self.vdt2 = g.zeros(device)
        # (u^{s-1}, u^s) at the start of each interval; None: the zero state of the first
        self.ckpt: list[tuple[torch.Tensor, torch.Tensor] | None] = []
        self.kept: list[torch.Tensor] = []  # checkpoint_every = 0: s_0 .. s_{nt-1}

    # ------------------------------------------------------------ forward
    def set_model(self, m_interior: torch.Tensor):
        g = self.grid
        g.interior(self.m).copy_(m_interior.detach())
        # only m's interior is read: vdt2's face halos take its periodic image
        api.prepare_vdt2_m(g, self.m, self.vdt2, self.dt)

    def forward(self, m_interior: torch.Tensor, checkpoints: bool = True) -> torch.Tensor:
        """Traces (nt, nrec) of the model m; keeps checkpoints for ``backward``."""
        g = self.grid
        self.set_model(m_interior)
        up, u, un = g.zeros(self.device), g.zeros(self.device), g.zeros(self.device)
        traces = torch.zeros((self.nt, self.nrec), dtype=torch.float32, device=self.device)
        self.ckpt = []
        if checkpoints and self.C == 0:
            if len(self.kept) != self.nt:
                self.kept = []
                torch.cuda.empty_cache()
                self.kept = [torch.empty(g.elems, dtype=torch.float32, device=self.device)
                             for _ in range(self.nt)]
            api.forward_keep(g, up, u, un, self.vdt2, self.sponge, self.nt, self.kept,
                             src=self.src, wavelet=self.w, rec_off=self.rec_off, traces=traces,
                             rec_plane=self.rec_plane)
            return traces
        self.kept = []
        step = self.C if self.C > 0 else self.nt
        for s in range(0, self.nt, step):  # one native loop per checkpoint interval
            e = min(s + step, self.nt)
            if checkpoints:
                self.ckpt.append((up.clone(), u.clone()) if s else None)
            up, u, un = api.forward_run(g, up, u, un, self.vdt2, self.sponge, e - s,
                                        src=self.src, wavelet=self.w[s:e],
                                        rec_off=self.rec_off, traces=traces[s:e],
                                        rec_plane=self.rec_plane)
        return traces

    @property
    def states(self) -> list[torch.Tensor]:
        """The wavefields of the last ``forward`` with checkpoint_every = 0, stepped again
        for each use (nt + 2 volumes): ``states[n]`` is u^n for n <= nt, the last is
        u^{-1} = 0.  Empty where the forward sweep kept nothing."""
        if not self.kept:
            return []
        g = self.grid
        u = [g.zeros(self.device) for _ in range(self.nt + 2)]
        for n in range(self.nt):
            api.step_fused(g, u[n - 1], u[n], u[n + 1], self.vdt2, self.sponge,
                           (self.src, float(self.w[n])))
        return u

    # ------------------------------------------------------------ adjoint
    def backward(self, res: torch.Tensor, want_grad_w: bool = False, scaled: bool = True,
                 want_lambda_src: bool = False):
        """grad_m (interior, float32) for trace residual ``res`` (nt, nrec) = dLoss/dtraces.

        ``scaled`` (default) runs the adjoint in b = vdt2 D lambda, where it is the
        forward update run backward in time (fd_adjoint_step_scaled); with
        ``want_grad_w`` it also returns dLoss/dw[n] = b^{n+1} at the source.
        ``scaled=False`` runs it in lambda itself (fd_adjoint_step); with
        ``want_lambda_src`` it also returns lambda^{n+1} at the source."""
        if scaled and want_lambda_src or not scaled and want_grad_w:
            raise ValueError("want_grad_w goes with scaled=True, want_lambda_src with False")
        g = self.grid
        nt, C = self.nt, self.C
        if not self.ckpt and not (C == 0 and self.kept):
            raise RuntimeError("backward needs a forward run with checkpoints")
        res = res.to(device=self.device, dtype=torch.float32).contiguous()
        if res.shape != (nt, self.nrec):
            raise ValueError(f"residual must be ({nt}, {self.nrec})")
        if scaled:
            return self._backward_scaled(res, want_grad_w)
        A = g.zeros(self.device)  # lambda^{n+2}
        B = g.zeros(self.device)  # lambda^{n+1}
        api.scatter_add(g, B, self.rec_off, res[nt - 1])
        gq = g.zeros(self.device)
        lam_src = torch.zeros(nt, dtype=torch.float32, device=self.device) if want_lambda_src else None
        for s, e, kept, last in self._segments(direct=True):
            for n in range(e - 1, s - 1, -1):
                if lam_src is not None:
                    api.record_receivers(g, B, self.src_off, lam_src[n:n + 1])
                if n == e - 1 and last is not None:
                    api.adjoint_step(g, A, B, A, self.vdt2, self.sponge, u_n=last, g_vdt2=gq,
                                     src=(self.src, float(self.w[n])))
                else:
                    api.grad_accumulate(g, B, kept[n - s], self.sponge, gq)
                    api.adjoint_step(g, A, B, A, self.vdt2, self.sponge)
                if n >= 1:
                    api.scatter_add(g, A, self.rec_off, res[n - 1])
                A, B = B, A
        gm = g.zeros(self.device)
        api.grad_finalize(g, gq, self.vdt2, self.dt, gm)
        out = g.interior(gm).clone()
        if want_lambda_src:
            return out, lam_src
        return out

    def _segments(self, direct: bool):
        """The segments of the reverse sweep, last first: (s, e, kept, last).  kept[i] =
        s_{s+i}, stored by the forward sweep or recomputed from the segment's checkpoint
        (into the same volumes for every segment), for s <= s + i < e, last None; or with
        ``direct`` for s + i < e - 1, and last = u^{e-1}, whose update is not needed."""
        if self.C == 0:
            yield 0, self.nt, self.kept, None
            return
        g = self.grid
        # only the interiors of the kept volumes are written and read; the wavefields'
        # zero halos are the Dirichlet boundary
        kept = [torch.empty(g.elems, dtype=torch.float32, device=self.device)
                for _ in range(min(self.C, self.nt) - direct)]
        field = [g.zeros(self.device) for _ in range(3 if len(kept) > 1 else len(kept))]
        # a few steps one by one only read the checkpoint; more than one do that on large
        # grids (a call costs 20 us of host time, copying the checkpoint 16 bytes a point)
        single = 3 if g.elems > 1 << 22 else 1
        for j in range(len(self.ckpt) - 1, -1, -1):
            s = j * self.C
            e = min(s + self.C, self.nt)
            n = e - s - direct
            if n <= single:
                up, u = self.ckpt[j] or (g.zeros(self.device), g.zeros(self.device))
                for i in range(n):
                    api.forward_keep(g, up, u, field[i], self.vdt2, self.sponge, 1, kept[i:i + 1],
                                     src=self.src, wavelet=self.w[s + i:s + i + 1])
                    up, u = u, field[i]
            else:
                for i in range(2):
                    if self.ckpt[j] is None:
                        field[i].zero_()
                    else:
                        field[i].copy_(self.ckpt[j][i])
                u = api.forward_keep(g, *field, self.vdt2, self.sponge, n, kept, src=self.src,
                                     wavelet=self.w[s:s + n])[1]
            yield s, e, kept, u if direct else None

    def _backward_scaled(self, res: torch.Tensor, want_grad_w: bool):
        g, nt = self.grid, self.nt
        A = g.zeros(self.device)  # b^{n+2}
        B = g.zeros(self.device)  # b^{n+1}
        api.scatter_add_scaled(g, B, self.rec_off, res[nt - 1], self.vdt2, self.sponge)
        gb = g.zeros(self.device)
        grad_w = torch.zeros(nt, dtype=torch.float32, device=self.device) if want_grad_w else None
        # a segment's last step on its state saves an update for two calls from here: worth it
        # where segments are short (us over 10 steps at 64^3 and 256^3, so / not so: C = 1 517
        # / 740 and 2425 / 3829, C = 2 485 / 507 and 2458 / 3014, C = 4 384 / 408 and 2373 / 2675)
        for s, e, kept, last in self._segments(direct=self.C <= DIRECT_STEPS):
            if last is not None:
                e -= 1
                if grad_w is not None:
                    api.record_receivers(g, B, self.src_off, grad_w[e:e + 1])
                inj = (self.rec_plane, res[e - 1]) if e and self.rec_plane is not None else None
                api.adjoint_step_scaled(g, A, B, A, self.vdt2, self.sponge, u_n=last, g_b=gb,
                                        src=(self.src, float(self.w[e])), res=inj)
                if e and inj is None:
                    api.scatter_add_scaled(g, A, self.rec_off, res[e - 1], self.vdt2, self.sponge)
                A, B = B, A
            if e == s:
                continue
            A, B = api.adjoint_run(g, A, B, self.vdt2, self.sponge, e - s, kept, gb,
                                   rec_off=self.rec_off, res=res[s:e],
                                   res0=res[s - 1] if s >= 1 else None, rec_plane=self.rec_plane,
                                   w_off=self.src_off if want_grad_w else None,
                                   w_out=grad_w[s:e] if want_grad_w else None)
        api.grad_finalize_scaled(g, gb, self.vdt2, self.dt, gb)
        out = g.interior(gb).clone()
        if want_grad_w:
            return out, grad_w
        return out


class FWIGrad(torch.autograd.Function):
    """traces = FWIGrad.apply(m, problem); m is the (nz, ny, nx) interior of the
    squared slowness on the device.  backward gives dLoss/dm."""

    @staticmethod
    def forward(ctx, m: torch.Tensor, problem: FWIProblem):
        ctx.problem = problem
        return problem.forward(m)

    @staticmethod
    def backward(ctx, grad_traces: torch.Tensor):
        return ctx.problem.backward(grad_traces), None


def misfit_gradient(problem: FWIProblem, m: torch.Tensor, obs: torch.Tensor):
    """J = 1/2 sum (traces - obs)^2 (accumulated in float64) and dJ/dm."""
    m = m.detach().clone().requires_grad_(True)
    tr = FWIGrad.apply(m, problem)
    r = tr - obs
    J = 0.5 * float((r.double() ** 2).sum().item())
    tr.backward(r)
    return J, m.grad
