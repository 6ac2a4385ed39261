"""Newton steps and adjoints from developed fields: a drop in its well, with walls a few nodes
thick, at dt L W towards 1 and (Cahn-Hilliard) dt M W^2 far above 4 kappa.  There the
spectrum is far better than the worst case of f'' says, and a polynomial chosen for that
would cost many times the products of the diagonal alone.

Counts.  The diagonal alone (point, and for Cahn-Hilliard 2x2 blocks), measured on these
steps: 21 to 51 products for Allen-Cahn, 396 and 390 iterations for Cahn-Hilliard.  A
product inside the polynomial costs a third to two thirds of one with its Gram-Schmidt
sweeps (eliminated Cahn-Hilliard, of half the unknowns: a third or less), so the bounds are
twice and three times those counts, where the worst case's interval takes four to ten and,
without a polynomial, 1.3 times of the dearer kind.  Roots: residual and energy balance are
the business of the other tests; here the oracle's Newton step bounds the root at one size."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import _abi as A
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, host, pair, rel_l2, rounded

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64


def drop(n, kappa):
    x = np.meshgrid(*[np.arange(k) - 0.5 * (k - 1) for k in reversed(n)], indexing="ij")
    return np.tanh((0.3 * min(n) - np.sqrt(sum(a * a for a in x))) / (2.0 * kappa) ** 0.5).ravel()


@pytest.mark.parametrize("n,kappa,dt,its", [((512, 512), 0.1, 0.99, 22), ((512, 512), 2.0, 0.9, 29),
                                            ((512, 512), 2.0, 0.99, 30), ((96, 96, 96), 0.1, 0.99, 26),
                                            ((96, 96, 96), 2.0, 0.9, 41), ((96, 96, 96), 2.0, 0.99, 41)])
def test_allen_cahn_drop(n, kappa, dt, its):
    announce("developed ac", n, kappa, dt)
    g, _ = pair(n, O.AC, O.F_SYM, F32, h=1.0, W=1.0, kappa=kappa, mob=1.0)
    U0 = dev(drop(n, kappa), F32)
    U = U0.clone()
    rep = S.newton_step(g, dt, U0, U)
    assert rep.converged and rep.gmres_its <= 2 * its, rep


@pytest.mark.parametrize("kappa,its", [(1.0, 126), (4.0, 317)])
def test_allen_cahn_half_developed(kappa, its):
    """Six time units after noise: pockets still below the wells, a few nodes wide, too small
    for a mode that f'' < 0 could carry.  The diagonal alone: 126 and 317 products."""
    announce("half developed ac", kappa)
    n = (96, 96, 96)
    g, _ = pair(n, O.AC, O.F_SYM, F32, h=1.0, W=1.0, kappa=kappa, mob=1.0)
    q, _ = pair(n, O.AC, O.F_SYM, F64, h=1.0, W=1.0, kappa=kappa, mob=1.0)
    u = dev(np.random.default_rng(3).uniform(-0.05, 0.05, 96**3), F64)
    S.step_explicit(q, u, 0.02, 300)
    U0 = u.to(F32)
    U = U0.clone()
    rep = S.newton_step(g, 0.99, U0, U)
    assert rep.converged and rep.gmres_its <= 2 * its, rep


@pytest.mark.parametrize("n,its", [((256, 256), 396), ((64, 64, 64), 390)])
def test_cahn_hilliard_drop_at_large_steps(n, its):
    announce("developed ch", n)
    g, _ = pair(n, O.CH, O.F_SYM, F32, h=1.0, W=1.0, kappa=2.0, mob=1.0)
    c = dev(drop(n, 2.0), F32)
    U0 = torch.cat([c, torch.zeros_like(c)])
    S.step_explicit(g, U0, 1e-6, 0)
    U = U0.clone()
    rep = S.newton_step(g, 50.0, U0, U)
    assert rep.converged and its < rep.gmres_its <= 3 * its, rep  # (a polynomial: cheaper products)


def test_cahn_hilliard_half_developed_at_a_large_step():
    """Thirty time units after noise, dt M W^2 / (4 kappa) = 5: the 2x2 blocks converge in 8
    corrections (none of them solved), the eliminated system alone not in 20."""
    announce("half developed ch")
    n, N = (256, 256), 256 * 256
    g, _ = pair(n, O.CH, O.F_SYM, F32, h=1.0, W=1.0, kappa=1.0, mob=1.0)
    q, _ = pair(n, O.CH, O.F_SYM, F64, h=1.0, W=1.0, kappa=1.0, mob=1.0)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    c = 0.05 * (2 * torch.rand(N, generator=gen, device="cuda", dtype=F64) - 1)
    u = torch.cat([c, torch.zeros_like(c)])
    S.step_explicit(q, u, 1.0 / 320, 9600)
    c = u[:N].to(F32)
    U0 = torch.cat([c, torch.zeros_like(c)])
    S.step_explicit(g, U0, 1e-6, 0)
    U = U0.clone()
    rep = S.newton_step(g, 20.0, U0, U)
    assert rep.converged and rep.newton_its <= 14, rep


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("model,n,dt", [(O.AC, (28, 24), 0.99), (O.AC, (10, 9, 8), 0.99), (O.AC, (28, 24), 3.0),
                                        (O.CH, (22, 18), 20.0), (O.CH, (7, 6, 8), 20.0)])
def test_roots_and_adjoints(model, n, dt, dtype):
    """Against the oracle's dense-LU step and adjoint.  Residuals of 1e-11 (FP64) and 1e-8 or
    the rounding floor (FP32) of the first; condition numbers of at most 1e3 (Allen-Cahn) and
    1e5 (Cahn-Hilliard, dt M kappa / h^4 = 40): 1e-8 and 1e-6, FP32 (floor 1e-7) 1e-4 and 1e-2."""
    announce("developed roots", model, n, dt, dtype)
    g, o = pair(n, model, O.F_SYM, dtype, h=1.0, W=1.0, kappa=2.0, mob=1.0, bc=O.NOFLUX)
    c = drop(n, 2.0)
    U0 = rounded(c if model == O.AC else O.explicit(o, np.concatenate([c, np.zeros_like(c)]), 1.0, 0), dtype)
    U = dev(U0, dtype)
    rep = S.newton_step(g, dt, dev(U0, dtype), U, S.newton_opts(rtol=1e-11 if dtype == F64 else 1e-8))
    assert rep.converged, rep
    Uo, conv, _, _ = O.newton_be(o, dt, U0, rtol=1e-13, maxit=40, solver=0)
    assert conv
    N = o.nnodes
    tol = {(O.AC, F64): 1e-8, (O.CH, F64): 1e-6, (O.AC, F32): 1e-4, (O.CH, F32): 1e-2}[model, dtype]
    assert rel_l2(host(U)[:N], Uo[:N]) < tol
    v = rounded(np.random.default_rng(4).standard_normal(o.ndof), dtype)
    Ur = rounded(Uo, dtype)
    ub, tb = torch.zeros(o.ndof, dtype=dtype, device="cuda"), torch.zeros(3, dtype=F64, device="cuda")
    S.vjp(g, A.VJP_NEWTON_STEP, dt, dev(Ur, dtype), dev(v, dtype), ub, tb)
    th, lam = O.newton_adjoint(o, dt, Ur, v, solver=0)
    assert rel_l2(host(ub), lam) < tol
