"""The limits a caller sets on the linear solves of a Newton step hold whatever the
preconditioner does inside a step of the solver."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import inputs as I
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, host, pair

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64


def stiff(n, dtype=F64, dt=0.5):
    # dt L kappa / h^2 = 75: products by the hundred with the diagonal alone
    g, o = pair(n, O.AC, O.F_SYM, dtype, h=0.1, W=1.0, kappa=1.5, mob=1.0, bc=O.NOFLUX)
    return g, o, dt, dev(I.uniform_field(n, -0.3, 0.3, seed=3), dtype)


@pytest.mark.parametrize("n", [(90, 70), (20, 18, 16)])
def test_gmres_max_its_counts_arnoldi_steps(n):
    """Eight steps are eight times the products of one."""
    announce("gmres_max_its", n)
    g, o, dt, U0 = stiff(n)
    its = []
    for limit in (1, 8):
        U = U0.clone()
        rep = S.newton_step(g, dt, U0, U, S.newton_opts(max_newton=1, gmres_max_its=limit, lin_rtol_min=1e-12,
                                                        lin_rtol_max=1e-12))
        its.append(rep.gmres_its)
    assert its[0] > 1 and its[1] == 8 * its[0]


@pytest.mark.parametrize("krylov", ["gmres", "cg"])
def test_linear_tolerance_is_the_callers(krylov):
    """Each correction is solved to clamp(0.1 ||R_k|| / ||R_0||, lin_rtol_min, lin_rtol_max),
    also where the Newton stop would be content with less: a field so small (1e-3) that the
    next residual is the linear solver's."""
    from paper_2601_06079_amd import _abi as A

    announce("linear tolerance", krylov)
    g, o, dt, _ = stiff((60, 50))
    U0 = dev(I.uniform_field((60, 50), -1e-3, 1e-3, seed=3), F64)
    U = U0.clone()
    rep = S.newton_step(g, dt, U0, U, S.newton_opts(rtol=1e-5, lin_rtol_min=1e-12, lin_rtol_max=1e-3,
                                                    krylov=A.KRYLOV_CG if krylov == "cg" else A.KRYLOV_GMRES))
    assert rep.converged and rep.newton_its == 2, rep
    r0, r1, r2 = rep.res_norm
    assert r1 / r0 <= 1.01e-3 and r2 / r1 <= 1.01 * 0.1 * r1 / r0
