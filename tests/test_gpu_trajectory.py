"""Explicit trajectories and their adjoint on both models, boundaries and dimensions, with
ragged lane groups and row blocks: the states against pf_step_explicit (bitwise), the
gradient against the oracle's discrete adjoint (FP64: the rounding of a few hundred
operations per node and step, held to 1e-10; FP32: 1e-5) and in segments (bitwise)."""
import ctypes as ct

import numpy as np
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import _abi as A
from paper_2601_06079_amd import inputs as I
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, host, pair, rel_l2, rounded

F32, F64 = torch.float32, torch.float64
STEPS = 4


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("bc", [O.PERIODIC, O.NOFLUX])
@pytest.mark.parametrize("model", [O.AC, O.CH])
@pytest.mark.parametrize("n", [(5, 4), (64, 11), (125, 18), (2, 2, 2), (21, 4, 3), (33, 7, 5), (63, 5, 6)])
def test_trajectory_and_adjoint(n, model, bc, dtype):
    announce("trajectory", n, model, bc, dtype)
    g, o = pair(n, model, O.F_SYM if model == O.AC else O.F_01, dtype, h=0.9, W=1.2, kappa=0.7, mob=1.1, bc=bc)
    N, dt = o.nnodes, 0.01
    c = I.uniform_field(n, -0.4, 0.4, seed=2, base=0.0 if model == O.AC else 0.5)
    U0 = rounded(c if model == O.AC else np.concatenate([c, np.zeros(N)]), dtype)
    states = torch.zeros((STEPS + 1, o.ndof), dtype=dtype, device="cuda")
    states[0].copy_(dev(U0, dtype))
    S.step_trajectory(g, states, dt)
    for k in range(STEPS):
        U = states[k].clone()
        S.step_explicit(g, U, dt, 1)
        assert torch.equal(U[:N], states[k + 1][:N])
        assert model == O.AC or k + 1 == STEPS or rel_l2(host(U)[N:], host(states[k + 1])[N:]) < 1e-5
    w = rounded(np.random.default_rng(3).standard_normal(o.ndof), dtype)
    w[N:] = 0.0
    ws = S.workspace(g, A.OP_VJP)
    lam, tb = dev(w, dtype), torch.zeros(3, dtype=F64, device="cuda")
    S.vjp_trajectory(g, states, lam, tb, dt, ws)
    tref, uref = O.explicit_adjoint(o, dt, STEPS, U0, w[:N])
    tol = 1e-10 if dtype == F64 else 1e-5
    assert rel_l2(host(lam)[:N], uref) < tol
    assert rel_l2(host(tb), tref) < tol
    lam2, tb2 = dev(w, dtype), torch.zeros(3, dtype=F64, device="cuda")
    S.vjp_trajectory(g, states[2:], lam2, tb2, dt, ws, begin=True, end=False)
    S.vjp_trajectory(g, states[:3], lam2, tb2, dt, ws, begin=False, end=True)
    assert torch.equal(lam, lam2) and torch.equal(tb, tb2)


def test_trajectory_argument_errors():
    """Refused before anything is enqueued (a context without a device)."""
    L = A.lib()
    C = ct.c_void_p()
    assert L.pf_create(A.HOST_ONLY, ct.byref(C)) == A.PF_OK
    fake = ct.c_void_p(0x1000)

    def call(dt=0.1, n=2, states=fake, flags=0, **kw):
        p = S.Problem(n=(8, 8), **kw).c()
        return (L.pf_step_explicit_trajectory(C, ct.byref(p), dt, n, states, None),
                L.pf_vjp_explicit_trajectory(C, ct.byref(p), dt, n, states, ct.c_void_p(0x2000), ct.c_void_p(0x3000),
                                             flags, ct.c_void_p(0x4000), None))

    assert call(dt=0.0) == (A.PF_EINVAL, A.PF_EINVAL)
    assert call(n=-1) == (A.PF_EINVAL, A.PF_EINVAL)
    assert call(states=None) == (A.PF_EINVAL, A.PF_EINVAL)
    assert call(model=A.COUPLED) == (A.PF_EUNSUPPORTED, A.PF_EUNSUPPORTED)
    assert call(mass=A.MASS_CONSISTENT) == (A.PF_EUNSUPPORTED, A.PF_EUNSUPPORTED)
    assert call(quad=A.QUAD_LOBATTO)[1] == A.PF_EUNSUPPORTED
    assert call(flags=4)[1] == A.PF_EINVAL
    assert L.pf_destroy(C) == A.PF_OK
