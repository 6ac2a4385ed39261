"""A fused step count that is set holds for runs of two steps too."""
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import _abi as A
from paper_2601_06079_amd import inputs as I
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, host, pair, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fuse,launches", [(0, 2), (1, 2), (2, 1)])
def test_two_steps(fuse, launches):
    """Launches alternate between the caller's array and the workspace: one launch leaves the
    result in the workspace (and copies it back), two leave the first step's state there."""
    announce("two steps", fuse)
    n = (130, 75)
    g, o = pair(n, O.AC, O.F_SYM, torch.float64, h=0.9, W=1.2, kappa=0.7, mob=1.1)
    c = I.uniform_field(n, -0.4, 0.4, seed=2)
    U = dev(c, torch.float64)
    ws = S.workspace(g, A.OP_STEP_EXPLICIT)
    try:
        S.tune_set(A.TUNE_STREAM2D_FUSE, fuse)
        S.step_explicit(g, U, 0.01, 2, ws)
    finally:
        S.tune_set(A.TUNE_STREAM2D_FUSE, 0)
    left = ws.view(torch.float64)[:o.nnodes]
    assert rel_l2(host(U), O.explicit(o, c, 0.01, 2)) < 1e-12
    assert rel_l2(host(left), O.explicit(o, c, 0.01, 2 if launches == 1 else 1)) < 1e-12
