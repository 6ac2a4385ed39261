"""The marching kernels of the weak forms without a direction (residual, explicit steps) at
the shapes where their layout can go wrong.  They run from 4 MiB a field in 2-D and from
2^19 nodes in 3-D (2^18 for all but the FP32 Cahn-Hilliard residual), so every shape here is
just above that, with the remainders in its short axes: lane groups of 64, 32, 21 and 16
columns that just fit or overflow, axes of two to seven nodes, row blocks and plane chunks
that do not divide.  Tolerances as for the other operator tests: a row sums a few hundred
products of rounded inputs, 1e-5 (FP32) and 1e-12 (FP64) of the result's norm."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import inputs as I
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, host, pair, rel_l2, rounded

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64
TOL = {F32: 1e-5, F64: 1e-12}


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("bc,quad", [(O.PERIODIC, 0), (O.NOFLUX, 0), (O.NOFLUX, 1)])
@pytest.mark.parametrize("n", [(2, 524300), (524300, 2), (62, 16913), (63, 16650), (125, 8390), (16400, 65),
                               (2, 2, 131100), (2, 740, 359), (19, 5, 5600), (20, 6, 4370), (30, 3, 5900),
                               (62, 4, 2120), (64, 7, 1181), (131, 2017, 2)])
def test_residual_and_step(n, bc, quad, dtype):
    announce("march shapes", n, bc, quad, dtype)
    assert np.prod(n) > (1 << 19) if len(n) == 3 else np.prod(n) * 4 >= 4 << 20
    c = I.uniform_field(n, -0.4, 0.4, seed=7, base=0.5)
    for model in (O.AC, O.CH):
        g, o = pair(n, model, O.F_01, dtype, h=0.7, W=1.3, kappa=0.9, mob=1.1, bc=bc)
        g.quad = o.quad = quad
        U = rounded(c if model == O.AC else np.concatenate([c, I.uniform_field(n, -0.5, 0.5, seed=8)]), dtype)
        assert rel_l2(host(S.residual(g, dev(U, dtype))), O.residual(o, U)) < TOL[dtype]
        if len(n) == 3:
            Ug = dev(U, dtype)
            S.step_explicit(g, Ug, 1e-3, 1)
            assert rel_l2(host(Ug), O.explicit(o, U, 1e-3, 1)) < TOL[dtype]
