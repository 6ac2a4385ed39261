"""FP32 weak forms: the coefficient of the stiffness is not rounded.  kappa is chosen so that
the folded number (kappa / 12 in 3-D, kappa / 3 in 2-D) lies nine tenths of the way to the
next FP32 one, 5.2e-8 off: with the nonlinear term all but switched off, every row would be
off by that factor.  Its projection on the FP64 rows is the mean of N rounding errors of at
most 3e-7 a row (a dozen operations) of random sign, 4e-10 for 5e5 rows and no more than ten
times that; held to 5e-9."""
import numpy as np
import pytest
import torch

from paper_2601_06079_amd import _abi as A
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kappa", [((90, 84, 80), 0.05), ((1100, 1000), 0.1)])
@pytest.mark.parametrize("bc", [A.PERIODIC, A.NOFLUX])
def test_stiffness_coefficient(n, kappa, bc):
    announce("stiffness coefficient", n, bc)
    folded = kappa / (12 if len(n) == 3 else 3)
    assert abs(float(np.float32(folded)) / folded - 1.0) > 5e-8
    kw = dict(n=n, model=A.ALLEN_CAHN, fe=A.F_SYM, bc=bc, h=1.0, W=1e-12, kappa=kappa, mobility=1.0)
    g = torch.Generator().manual_seed(1)
    U = torch.rand(int(np.prod(n)), generator=g, dtype=torch.float32).cuda()
    r32 = S.residual(S.Problem(dtype=torch.float32, **kw), U).double()
    r64 = S.residual(S.Problem(dtype=torch.float64, **kw), U.double())
    assert abs((((r32 - r64) * r64).sum() / (r64 * r64).sum()).item()) < 5e-9
