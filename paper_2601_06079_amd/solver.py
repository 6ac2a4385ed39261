"""Torch-facing wrappers of the C ABI: same names as include/pf.h, no arithmetic.

Tensors must be contiguous CUDA (HIP) tensors of the problem's dtype.  Every
call is enqueued on torch's current stream.
"""
from __future__ import annotations

import ctypes as ct
from dataclasses import dataclass, field, replace

import torch

from . import _abi as A


@dataclass
class Problem:
    """Problem statement (see pf_problem in include/pf.h)."""
    n: tuple
    model: int = A.ALLEN_CAHN
    fe: int = A.F_SYM
    dtype: torch.dtype = torch.float32
    h: float = 1.0
    W: float = 1.0
    kappa: float = 1.0
    mobility: float = 1.0
    bc: int = A.PERIODIC
    mobility_eta: float = 0.0  # coupled model: M_eta
    mass: int = A.MASS_LUMPED  # MASS_CONSISTENT: Gauss-integrated mass (implicit path)
    nfields: int = 1  # GRAIN: order parameters
    gamma: float = 1.5  # GRAIN: pair coupling
    quad: int = A.QUAD_GAUSS  # QUAD_LOBATTO: nodal quadrature

    @property
    def dim(self):
        return len(self.n)

    @property
    def nnodes(self):
        N = 1
        for v in self.n:
            N *= int(v)
        return N

    @property
    def ndof(self):
        if self.model == A.GRAIN:
            return int(self.nfields) * self.nnodes
        return _FIELDS.get(self.model, 1) * self.nnodes

    def c(self) -> A.pf_problem:
        n = self.n
        d = len(n)
        n3 = _N3(int(n[0]), int(n[1]), int(n[2]) if d > 2 else 1) if d in (2, 3) else _N3(*(int(v) for v in n), 1, 1)
        return A.pf_problem(d, self.bc, self.model, self.fe, A.F64 if self.dtype == torch.float64 else A.F32,
                            int(self.mass), n3, float(self.h), float(self.W), float(self.kappa),
                            float(self.mobility), float(self.mobility_eta), int(self.nfields), int(self.quad),
                            float(self.gamma))


_FIELDS = {A.CAHN_HILLIARD: 2, A.COUPLED: 3}
_N3 = ct.c_int64 * 3


# A small call's kernels take 8 us and its wrapper took 8 as well: the current device's
# stream and context are looked up by index, without stream and device objects, and the
# sizes worked out once a call (three operators at 1001 x 777: 33 us before).
def _stream():
    return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())


def _ctx():
    device = torch.cuda.current_device()
    return A._ctxs.get(device) or A.ctx(device)


def _ptr(t: torch.Tensor, p: Problem = None, n: int = None, name="tensor"):
    if not t.is_cuda:
        raise ValueError(f"{name} must be a device tensor")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if p is not None and t.dtype != p.dtype:
        raise ValueError(f"{name} has dtype {t.dtype}, problem says {p.dtype}")
    if n is not None and t.numel() != n:
        raise ValueError(f"{name} has {t.numel()} elements, expected {n}")
    return t.data_ptr()


def workspace(p: Problem, op: int, device=None) -> torch.Tensor:
    nb = ct.c_size_t(0)
    A.check(A.lib().pf_workspace_size(A.ctx(device), ct.byref(p.c()), op, ct.byref(nb)))
    return torch.empty(max(int(nb.value), 8), dtype=torch.uint8,
                       device=device or torch.device("cuda"))


def residual(p: Problem, U: torch.Tensor, out: torch.Tensor = None) -> torch.Tensor:
    r = torch.empty_like(U) if out is None else out
    nd = p.ndof
    A.check(A.lib().pf_residual(_ctx(), ct.byref(p.c()), _ptr(U, p, nd, "U"), _ptr(r, p, nd, "r"), None,
                                _stream()))
    return r


def step_explicit(p: Problem, U: torch.Tensor, dt: float, nsteps: int,
                  ws: torch.Tensor = None) -> torch.Tensor:
    """nsteps explicit steps in place on U; returns U."""
    if ws is None:
        ws = workspace(p, A.OP_STEP_EXPLICIT, U.device)
    A.check(A.lib().pf_step_explicit(_ctx(), ct.byref(p.c()), float(dt), int(nsteps),
                                     _ptr(U, p, p.ndof, "U"), ws.data_ptr(), _stream()))
    return U


def energy(p: Problem, U: torch.Tensor, ws: torch.Tensor = None,
           out: torch.Tensor = None) -> torch.Tensor:
    """Device tensor [E_h, sum m c] (float64)."""
    if ws is None:
        ws = workspace(p, A.OP_ENERGY, U.device)
    if out is None:
        out = torch.empty(2, dtype=torch.float64, device=U.device)
    A.check(A.lib().pf_energy(_ctx(), ct.byref(p.c()), _ptr(U, p, p.ndof, "U"), out.data_ptr(), ws.data_ptr(),
                              _stream()))
    return out


def jvp(p: Problem, inv_dt: float, U: torch.Tensor, v: torch.Tensor,
        out: torch.Tensor = None) -> torch.Tensor:
    Jv = torch.empty_like(U) if out is None else out
    nd = p.ndof
    A.check(A.lib().pf_jvp(_ctx(), ct.byref(p.c()), float(inv_dt), _ptr(U, p, nd, "U"), _ptr(v, p, nd, "v"),
                           _ptr(Jv, p, nd, "Jv"), _stream()))
    return Jv


def newton_opts(**kw) -> A.pf_newton_opts:
    o = A.pf_newton_opts()
    A.lib().pf_newton_default_opts(ct.byref(o))
    for k, v in kw.items():
        setattr(o, k, v)
    return o


@dataclass
class NewtonReport:
    newton_its: int
    gmres_its: int
    converged: bool
    reason: int
    res_norm: list = field(default_factory=list)


def newton_step(p: Problem, dt: float, U_old: torch.Tensor, U: torch.Tensor, opts=None,
                ws: torch.Tensor = None, raise_on_noconv: bool = False) -> NewtonReport:
    """One backward-Euler step in place on U (initial guess on entry)."""
    if ws is None:
        ws = workspace(p, A.OP_NEWTON, U.device)
    o = opts if opts is not None else newton_opts()
    rep = A.pf_newton_report()
    st = A.lib().pf_newton_step(A.ctx(), ct.byref(p.c()), float(dt), _ptr(U_old, p, p.ndof, "U_old"),
                                _ptr(U, p, p.ndof, "U"), ct.byref(o), ct.byref(rep),
                                ct.c_void_p(ws.data_ptr()), _stream())
    allow = () if raise_on_noconv else (A.PF_ENOCONV, A.PF_ENONFINITE)
    A.check(st, allow=allow)
    k = rep.newton_its
    return NewtonReport(k, rep.gmres_its, bool(rep.converged), rep.reason,
                        [rep.res_norm[i] for i in range(min(k, 32) + 1)])


def _check_theta(theta_bar: torch.Tensor):
    if theta_bar.dtype != torch.float64 or theta_bar.numel() != 3 or not theta_bar.is_contiguous():
        raise ValueError("theta_bar must be a contiguous float64 tensor of 3 entries")


def vjp(p: Problem, kind: int, dt: float, U: torch.Tensor, vbar: torch.Tensor,
        Ubar: torch.Tensor, theta_bar: torch.Tensor, ws: torch.Tensor = None,
        U_old: torch.Tensor = None):
    """Accumulate vector-Jacobian products into Ubar and theta_bar (float64[3], on the
    device or, making the call host-synchronous, on the host).  U_old (VJP_RESIDUAL
    only) selects the backward-Euler residual M (U - U_old)/dt + r(U)."""
    if ws is None:
        ws = workspace(p, A.OP_VJP, U.device)
    _check_theta(theta_bar)
    flags = 0 if theta_bar.is_cuda else A.VJP_THETA_HOST
    uold = None if U_old is None else _ptr(U_old, p, p.ndof, "U_old")
    A.check(A.lib().pf_vjp(A.ctx(), ct.byref(p.c()), int(kind), float(dt), _ptr(U, p, p.ndof, "U"),
                           uold, _ptr(vbar, p, None, "vbar"), _ptr(Ubar, p, None, "Ubar"),
                           ct.c_void_p(theta_bar.data_ptr()), flags, ct.c_void_p(ws.data_ptr()),
                           _stream()))


def step_trajectory(p: Problem, states: torch.Tensor, dt: float):
    """states[1:] from states[0] by single explicit steps, every state kept
    (states: steps + 1 rows of ndof)."""
    n = states.shape[0] - 1
    A.check(A.lib().pf_step_explicit_trajectory(A.ctx(), ct.byref(p.c()), float(dt), n,
                                                _ptr(states, p, (n + 1) * p.ndof, "states"), _stream()))


def vjp_trajectory(p: Problem, states: torch.Tensor, lam: torch.Tensor, theta_bar: torch.Tensor, dt: float,
                   ws: torch.Tensor, begin: bool = True, end: bool = True):
    """Adjoint of step_trajectory: lam (dO/d last state) becomes dO/d states[0]; the
    gradient of theta accumulates in ws from begin and is added to theta_bar (float64[3], on
    the device) at end."""
    _check_theta(theta_bar)
    n = states.shape[0] - 1
    flags = (A.VJP_BEGIN if begin else 0) | (A.VJP_END if end else 0)
    A.check(A.lib().pf_vjp_explicit_trajectory(A.ctx(), ct.byref(p.c()), float(dt), n,
                                               _ptr(states, p, (n + 1) * p.ndof, "states"),
                                               _ptr(lam, p, p.ndof, "lam"), _ptr(theta_bar, None, 3, "theta_bar"),
                                               flags, ct.c_void_p(ws.data_ptr()), _stream()))


def launch_shape(p: Problem):
    """(steps fused per launch, rows per wave, prefetch depth) that step_explicit
    uses for the 2-D problem p."""
    ks, ty, dp = ct.c_int(0), ct.c_int(0), ct.c_int(0)
    A.check(A.lib().pf_launch_shape(A.ctx(), ct.byref(p.c()), ct.byref(ks), ct.byref(ty), ct.byref(dp)))
    return int(ks.value), int(ty.value), int(dp.value)


def tune_set(key: int, value: int):
    A.check(A.lib().pf_tune_set(int(key), int(value)))


def tune_get(key: int) -> int:
    v = ct.c_int(0)
    A.check(A.lib().pf_tune_get(int(key), ct.byref(v)))
    return int(v.value)


# ---------------------------------------------------------------------------
class CheckpointedRun(torch.autograd.Function):
    """U_N = S^N(U_0; theta) for one problem, explicit (Eq. 12) or backward-Euler
    Newton steps (Eqs. 13-14), with a hand-written adjoint (Supp. Note 2,
    Eqs. II.5-II.6).

    theta = (mobility, kappa, W) as a float64 tensor of 3.  Forward keeps a
    snapshot every `every` steps (explicit runs with keep also the last segment's
    states, which the first backward takes over as its buffer); backward walks the
    segments in reverse, recomputes each segment's states from its snapshot (bitwise
    the forward's: every kernel is deterministic, and both passes advance with the
    same launches: fused launches are bitwise single steps on periodic grids, and
    no-flux grids, where a fused stage rounds the reflected rows differently, take
    single-step launches in the forward pass too) and applies the step adjoint of the
    library (the explicit trajectory's adjoint, or the transposed Newton solve at each
    root), accumulating the gradient of theta in FP64.  For Cahn-Hilliard explicit
    runs only the c plane of U_N is differentiated (mu is recomputed from c).
    """

    @staticmethod
    def forward(ctx, theta, U0, p, dt, nsteps, every, implicit, opts, keep=True):
        if nsteps % every:
            raise ValueError("nsteps must be a multiple of the checkpoint interval")
        th = theta.detach().to("cpu", torch.float64).numpy()
        q = replace(p, mobility=float(th[0]), kappa=float(th[1]), W=float(th[2]))
        U = U0.detach().clone()
        # the library's trajectory calls: both models, fields below 2 GiB
        es = torch.empty((), dtype=q.dtype).element_size()
        traj = not implicit and q.model in (A.ALLEN_CAHN, A.CAHN_HILLIARD) and q.nnodes * es < 1 << 31
        nseg = nsteps // every
        kept = 1 if traj and nseg and keep else 0  # segments whose states are kept
        snaps = []
        if nseg > kept:
            ws = workspace(q, A.OP_NEWTON if implicit else A.OP_STEP_EXPLICIT, U.device)
        single = q.bc == A.NOFLUX  # match the single-step recomputation bitwise
        for _ in range(nseg - kept):
            snaps.append(U.clone())
            if single:
                for _ in range(every):
                    _advance(q, U, dt, 1, implicit, opts, ws)
            else:
                _advance(q, U, dt, every, implicit, opts, ws)
        ctx.last = []
        if kept:
            _ptr(U, q, q.ndof, "U")
            snaps.append(U.clone())
            last = torch.empty((every + 1, U.numel()), dtype=q.dtype, device=U.device)
            last[0].copy_(U.view(-1))
            step_trajectory(q, last, dt)
            U.view(-1).copy_(last[every])
            ctx.last.append(last)
        ctx.q, ctx.dt, ctx.every, ctx.implicit, ctx.opts = q, dt, every, implicit, opts
        ctx.snaps, ctx.theta_device, ctx.traj = snaps, theta.device, traj
        return U

    @staticmethod
    def backward(ctx, gU):
        q, dt, every, implicit = ctx.q, ctx.dt, ctx.every, ctx.implicit
        lam = gU.detach().to(q.dtype).contiguous().clone().view(-1)
        N = q.nnodes
        if q.model == A.CAHN_HILLIARD and not implicit:
            lam[N:] = 0
        tb = torch.zeros(3, dtype=torch.float64, device=lam.device)
        vws = workspace(q, A.OP_VJP, lam.device)
        if ctx.traj:
            top = len(ctx.snaps) - 1
            try:
                states = ctx.last.pop()  # a later backward of the same graph forms it again
                formed = top
            except IndexError:
                states = torch.empty((every + 1, lam.numel()), dtype=q.dtype, device=lam.device)
                formed = top + 1
            for i in range(top, -1, -1):
                if i < formed:
                    states[0].copy_(ctx.snaps[i].view(-1))
                    step_trajectory(q, states, dt)
                vjp_trajectory(q, states, lam, tb, dt, vws, begin=i == top, end=i == 0)
            return tb.to(ctx.theta_device), lam.view(gU.shape), None, None, None, None, None, None, None
        ws = workspace(q, A.OP_NEWTON if implicit else A.OP_STEP_EXPLICIT, lam.device)
        seg = torch.empty((every + 1, lam.numel()), dtype=q.dtype, device=lam.device)
        Ubar = torch.empty_like(lam)
        kind = A.VJP_NEWTON_STEP if implicit else A.VJP_EXPLICIT_STEP
        for snap in reversed(ctx.snaps):
            seg[0].copy_(snap.view(-1))
            for k in range(every):  # seg[k + 1] = S(seg[k])
                seg[k + 1].copy_(seg[k])
                _advance(q, seg[k + 1], dt, 1, implicit, ctx.opts, ws)
            for k in reversed(range(every)):
                # explicit: VJP of the step taken from seg[k]; implicit: at its root seg[k + 1]
                Ubar.zero_()
                vjp(q, kind, dt, seg[k + 1] if implicit else seg[k], lam, Ubar, tb, vws)
                lam, Ubar = Ubar, lam
        return tb.to(ctx.theta_device), lam.view(gU.shape), None, None, None, None, None, None, None


def _advance(q, U, dt, nsteps, implicit, opts, ws):
    if not implicit:
        step_explicit(q, U, dt, nsteps, ws)
        return
    Uold = torch.empty_like(U)
    for _ in range(nsteps):
        Uold.copy_(U)
        newton_step(q, dt, Uold, U, opts, ws, raise_on_noconv=True)


def checkpointed_run(theta, U0, p, dt, nsteps, every=100, implicit=False, opts=None):
    """Differentiable run of nsteps steps of problem p (see CheckpointedRun)."""
    keep = torch.is_grad_enabled() and (theta.requires_grad or U0.requires_grad)
    return CheckpointedRun.apply(theta, U0, p, dt, nsteps, every, implicit, opts, keep)
