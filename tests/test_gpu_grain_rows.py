"""Explicit grain growth on grids that take each kind of chunk: one row a wave, one wave
per SIMD, several, more than stay resident.  Against the FP64 oracle with the bounds of
the other grain tests: 2e-6 (FP32) and 1e-12 (FP64) per step of fields of order one."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import _abi as A
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, host, rounded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n,p,bc", [((96, 96), 8, O.PERIODIC), ((70, 5), 2, O.NOFLUX), ((420, 401), 6, O.NOFLUX),
                                    ((1010, 607), 8, O.PERIODIC), ((1300, 1201), 3, O.PERIODIC)])
def test_steps_at_every_chunk_length(n, p, bc, dtype):
    announce("grain rows", n, p, bc, dtype)
    g = S.Problem(n=n, model=A.GRAIN, dtype=dtype, h=0.9, kappa=0.8, mobility=1.2,
                  bc=A.NOFLUX if bc == O.NOFLUX else A.PERIODIC, nfields=p, gamma=1.4)
    o = O.GrainProblem(n, p=p, bc=bc, h=0.9, L=1.2, kappa=0.8, gamma=1.4)
    U = rounded(np.random.default_rng(p).uniform(-0.1, 1.1, o.ndof), dtype)
    Ug = dev(U, dtype)
    S.step_explicit(g, Ug, 0.02, 2)
    assert np.abs(host(Ug) - O.gg_explicit(o, U, 0.02, 2)).max() <= (1e-12 if dtype == torch.float64 else 2e-6) * 2
