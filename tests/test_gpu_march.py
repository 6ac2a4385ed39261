"""The marching stencil kernels (march.hpp) at the sizes where their work layout can go
wrong: lane groups of 64, 32, 21 and 16 columns that just fit or just overflow, row
blocks and plane chunks with remainders, both row counts per lane, both boundaries and
both quadratures, against the oracle.  Tolerances: a row sums a few hundred products of
rounded inputs, so 1e-5 (FP32) and 1e-12 (FP64) of the result's norm, as for the other
operator tests."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import _abi as A
from paper_2601_06079_amd import inputs as I
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, host, pair, rel_l2, rounded

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64
TOL = {F32: 1e-5, F64: 1e-12}


def case(n, model, bc, quad, dtype):
    g, o = pair(n, model, O.F_01, dtype, h=0.7, W=1.3, kappa=0.9, mob=1.1, bc=bc)
    g.quad = o.quad = quad
    c = I.uniform_field(n, -0.4, 0.4, seed=7, base=0.5)
    U = c if model == O.AC else np.concatenate([c, I.uniform_field(n, -0.5, 0.5, seed=8)])
    return g, o, rounded(U, dtype)


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("quad", [0, 1])
@pytest.mark.parametrize("bc", [O.PERIODIC, O.NOFLUX])
@pytest.mark.parametrize("n", [(2, 2), (62, 9), (63, 8), (125, 33),
                               (2, 2, 2), (19, 5, 3), (20, 6, 7), (30, 3, 4), (62, 4, 2), (64, 7, 9)])
def test_residual_and_step(n, bc, quad, dtype):
    """Residual of both models and (3-D) three explicit steps of each."""
    announce("march", n, bc, quad, dtype)
    for model in (O.AC, O.CH):
        g, o, U = case(n, model, bc, quad, dtype)
        assert rel_l2(host(S.residual(g, dev(U, dtype))), O.residual(o, U)) < TOL[dtype]
        if len(n) == 3:
            Ug = dev(U, dtype)
            S.step_explicit(g, Ug, 1e-3, 3)
            assert rel_l2(host(Ug), O.explicit(o, U, 1e-3, 3)) < TOL[dtype]


@pytest.mark.parametrize("bc,quad,dtype", [(O.PERIODIC, 0, F32), (O.NOFLUX, 0, F32), (O.PERIODIC, 0, F64),
                                           (O.NOFLUX, 1, F32)])
def test_many_nodes_per_lane(bc, quad, dtype):
    """Above 2^20 nodes a lane carries four rows: ragged 3-D grid, residual and one step."""
    n = (131, 102, 81)
    announce("march large", n, bc, quad, dtype)
    g, o, U = case(n, O.CH, bc, quad, dtype)
    assert rel_l2(host(S.residual(g, dev(U, dtype))), O.residual(o, U)) < TOL[dtype]
    Ug = dev(U, dtype)
    S.step_explicit(g, Ug, 1e-3, 1)
    assert rel_l2(host(Ug), O.explicit(o, U, 1e-3, 1)) < TOL[dtype]


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("n,bc,quad", [((14, 141, 135), O.NOFLUX, 0), ((19, 120, 118), O.PERIODIC, 0),
                                       ((30, 99, 90), O.NOFLUX, 1), ((62, 71, 62), O.NOFLUX, 0),
                                       ((64, 65, 64), O.PERIODIC, 1), ((64, 64, 64), O.NOFLUX, 0),
                                       ((1031, 1021), O.NOFLUX, 0), ((1025, 1030), O.PERIODIC, 1)])
def test_just_above_the_node_kernels(n, bc, quad, dtype):
    """The smallest grids that march, one lane-group count each (64^3: the largest that
    does not); residual and, in 3-D, two explicit steps."""
    announce("march from", n, bc, quad, dtype)
    for model in (O.AC, O.CH):
        g, o, U = case(n, model, bc, quad, dtype)
        assert rel_l2(host(S.residual(g, dev(U, dtype))), O.residual(o, U)) < TOL[dtype]
        if len(n) == 3:
            Ug = dev(U, dtype)
            S.step_explicit(g, Ug, 1e-3, 2)
            assert rel_l2(host(Ug), O.explicit(o, U, 1e-3, 2)) < TOL[dtype]
