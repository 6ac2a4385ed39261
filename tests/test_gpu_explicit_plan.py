"""The 2-D explicit runs' launch plan: step counts that leave every remainder (launches of
unequal lengths, odd and even numbers of them) on grids that take each kind of plan (one
row group, fewer waves than SIMDs, one and several rounds, shared and recomputed seams),
against the same run in single steps.  Periodic grids: the same bits (each node's
arithmetic does not depend on the launch shape).  No-flux: a fused stage evaluates
reflected ghost rows, which differ from the inner rows in the last place: over 13 steps
16 units in the last place of the field."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import _abi as A
from paper_2601_06079_amd import inputs as I
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, pair, rounded

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("bc,quad", [(O.PERIODIC, 0), (O.NOFLUX, 0), (O.PERIODIC, 1)])
@pytest.mark.parametrize("model", [O.AC, O.CH])
@pytest.mark.parametrize("n", [(5, 3), (61, 130), (500, 90), (640, 700)])
def test_plan_against_single_steps(n, model, bc, quad, dtype):
    announce("explicit plan", n, model, bc, quad, dtype)
    g, o = pair(n, model, O.F_01, dtype, h=1.0, W=1.0, kappa=0.7, mob=1.0, bc=bc)
    g.quad = quad
    c = I.uniform_field(n, -0.3, 0.3, seed=5, base=0.5)
    U = rounded(c if model == O.AC else np.concatenate([c, np.zeros_like(c)]), dtype)
    for steps in (1, 2, 3, 4, 5, 7, 8, 10, 13):
        a, b = dev(U, dtype), dev(U, dtype)
        S.step_explicit(g, a, 0.005, steps)
        try:
            S.tune_set(A.TUNE_STREAM2D_FUSE, 1)
            S.step_explicit(g, b, 0.005, steps)
        finally:
            S.tune_set(A.TUNE_STREAM2D_FUSE, 0)
        N = o.nnodes
        if bc == O.PERIODIC:
            assert torch.equal(a[:N], b[:N]), steps
        else:
            eps = torch.finfo(dtype).eps
            assert (a[:N] - b[:N]).abs().max() <= 16 * eps * b[:N].abs().max(), steps


@pytest.mark.parametrize("dtype", [F32, F64])
def test_batch_rows_do_not_matter(dtype):
    """A batch large enough for chunks other than the shortest: the same bits as with 8 rows."""
    announce("batch rows", dtype)
    from paper_2601_06079_amd import batch as B

    sizes = [(130 + 24 * i, 500 - 20 * i) for i in range(16)]
    th = [(1.0 + 0.01 * i, 0.7, 1.0) for i in range(16)]
    out = []
    for ty in (0, 8):
        b = B.Batch(sizes, th, 0.05, dtype=dtype, ty=ty)
        assert (b.info.ty > 8) == (ty == 0)
        U = b.empty()
        for i, v in enumerate(b.views(U)):
            v.copy_(dev(I.uniform_field(sizes[i], -0.3, 0.3, seed=i, base=0.0), dtype).view_as(v))
        b.step(U, 6)
        out.append([v.clone() for v in b.views(U)])
    for x, y in zip(*out):
        assert torch.equal(x, y)
