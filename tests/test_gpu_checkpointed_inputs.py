"""Explicit checkpointed runs: what they accept (a field of the problem's type whose copy is
contiguous, in any shape of its size), the memory a run without a gradient
takes, and a second backward of one graph (bitwise the first)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2601_06079_amd import inputs as I
from paper_2601_06079_amd import solver as S
from tests.gpu_util import announce, dev, host, pair, rel_l2, rounded

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64
THETA = [1.1, 0.7, 1.2]


def problem(n=(24, 20), dtype=F64, model=O.AC):
    g, o = pair(n, model, O.F_SYM, dtype, h=0.9, W=1.2, kappa=0.7, mob=1.1)
    c = I.uniform_field(n, -0.4, 0.4, seed=2)
    return g, o, rounded(c, dtype)


def theta():
    return torch.tensor(THETA, dtype=F64, requires_grad=True)


@pytest.mark.parametrize("nsteps,every", [(4, 4), (6, 2)])
def test_what_is_refused(nsteps, every):
    announce("checkpointed inputs", nsteps, every)
    g, o, c = problem()
    for bad in (dev(c, F32), dev(c, F64)[:-1], torch.as_tensor(c), dev(c, F64).view(20, 24).t()):
        with pytest.raises((ValueError, TypeError)):
            S.checkpointed_run(theta(), bad, g, 0.01, nsteps, every)


@pytest.mark.parametrize("nsteps,every", [(4, 4), (6, 2)])
def test_field_of_another_shape(nsteps, every):
    announce("checkpointed shape", nsteps, every)
    g, o, c = problem()
    w = dev(np.random.default_rng(1).standard_normal(o.nnodes), F64)
    out = []
    for shape in ((o.nnodes,), (20, 24), (1, 20, 24), "strided"):
        th, u = theta(), dev(c, F64)
        if shape == "strided":
            shape, u = (o.nnodes,), u.repeat_interleave(2)[::2]
        u = u.view(shape).requires_grad_(True)
        U = S.checkpointed_run(th, u, g, 0.01, nsteps, every)
        assert U.shape == shape
        (U * w.view(shape)).sum().backward()
        out.append((U.detach().reshape(-1), u.grad.reshape(-1), th.grad))
    for a in out[1:]:
        assert all(torch.equal(x, y) for x, y in zip(a, out[0]))
    tref, uref = O.explicit_adjoint(o, 0.01, nsteps, c, host(w))
    assert rel_l2(host(out[0][1]), uref) < 1e-10 and rel_l2(host(out[0][2]), tref) < 1e-10


@pytest.mark.parametrize("model", [O.AC, O.CH])
def test_second_backward(model):
    announce("checkpointed twice", model)
    g, o, c = problem(model=model)
    U0 = c if model == O.AC else np.concatenate([c, np.zeros_like(c)])
    w = dev(np.random.default_rng(1).standard_normal(o.ndof), F64)
    th, u = theta(), dev(U0, F64).requires_grad_(True)
    U = S.checkpointed_run(th, u, g, 0.01, 6, 2)
    a = torch.autograd.grad((U * w).sum(), (th, u), retain_graph=True)
    b = torch.autograd.grad((U * w).sum(), (th, u))
    assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_run_without_a_gradient_keeps_no_states():
    """50 steps in one segment: 51 states of 2 MB if they were kept, two or three if not."""
    announce("checkpointed no grad")
    g, o, c = problem((512, 512), F64)
    U0 = dev(c, F64)
    with torch.no_grad():
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        S.checkpointed_run(theta(), U0, g, 0.01, 50, 50)
        assert torch.cuda.max_memory_allocated() - before < 6 * U0.numel() * 8
