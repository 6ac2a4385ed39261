"""The elastic solver's kernels at the sizes where they branch: the eigenstrain load
with the flat parts of its profile skipped, and the V-cycle whose 3-D coarse end runs
in one workgroup, both against the FP64 oracle.

Tolerances.  The skipped part of the profile differs from its limit by less than
1 - tanh 20 = 8e-18 of the amplitude, so the load keeps the bounds of the evaluated
one: 1e-13 (FP64) and 1e-6 (FP32) of the largest entry.  Solves to rtol: within a
condition number (about 1e3 for the preconditioned operator and its norms) of it.
"""
import numpy as np
import pytest
import torch

import oracle as O
from tests.gpu_util import announce, host, rel_l2
from paper_2601_06079_amd import _abi as A
from paper_2601_06079_amd import elastic as EL

pytestmark = pytest.mark.gpu


def pair(n, dtype, **kw):
    d = dict(h=100.0 / (max(n) - 1), E=22.5, nu=0.3, m=0.01, a=20.0, l=0.5)
    d.update(kw)
    return EL.ElasticProblem(n=tuple(n), dtype=dtype, **d), O.ElasticProblem(n=tuple(n), **d)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("a,l", [(40.0, 3.0), (40.0, -3.0), (40.0, 0.0), (40.0, 1e6), (-5.0, 2.0), (-60.0, 2.0),
                                 (0.0, 1.0), (150.0, 2.0), (20.0, 1e-300)])
@pytest.mark.parametrize("n", [(21, 34), (9, 13, 6)])
def test_load_where_the_profile_is_flat(n, a, l, dtype):
    announce("el_rhs flat", n, a, l, dtype)
    g, o = pair(n, dtype, a=a, l=l)
    f, ref = host(EL.el_rhs(g)), O.el_rhs(o)
    tol = 1e-13 if dtype == torch.float64 else 1e-6
    scale = max(np.abs(ref).max(), 22.5 * 0.01 * g.h ** (g.dim - 1) * 1e-3)
    assert np.abs(f - ref).max() <= tol * scale


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [(5, 5, 5), (9, 5, 7), (17, 17, 17), (33, 17, 9), (65, 9, 5), (5, 33, 65)])
def test_coarse_block_is_the_cycle(n, dtype):
    """The default 3-D cycle (coarse end in one block where it fits) against every
    level launched separately: the same iterations (to one) and solution."""
    announce("el coarse block 3-D", n, dtype)
    g, o = pair(n, dtype)
    rtol = 1e-11 if dtype == torch.float64 else 1e-5
    L = A.lib()
    u, rep = EL.el_solve(g, rtol=rtol)
    try:
        assert L.pf_tune_set(EL.TUNE_EL_MG, 2) == A.PF_OK
        us, reps = EL.el_solve(g, rtol=rtol)
    finally:
        L.pf_tune_set(EL.TUNE_EL_MG, 0)
    assert rep.converged and reps.converged and rep.levels == reps.levels
    assert abs(rep.iterations - reps.iterations) <= 1
    ref, _ = O.el_solve(o, rtol=1e-13)
    assert rel_l2(host(u), ref) < 1e3 * rtol and rel_l2(host(us), ref) < 1e3 * rtol
