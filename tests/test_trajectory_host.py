"""Argument checks of the trajectory calls' wrappers (no device needed)."""
import pytest
import torch

from paper_2601_06079_amd import solver as S


@pytest.mark.parametrize("theta_bar", [torch.zeros(3, dtype=torch.float32), torch.zeros(2, dtype=torch.float64),
                                       torch.zeros(6, dtype=torch.float64)[::2]])
def test_trajectory_theta_bar_is_three_doubles(theta_bar):
    """The library adds three doubles there: nothing smaller may reach it."""
    p = S.Problem(n=(8, 8))
    states, lam = torch.zeros((3, 64), dtype=p.dtype), torch.zeros(64, dtype=p.dtype)
    with pytest.raises(ValueError, match="theta_bar must be a contiguous float64 tensor of 3"):
        S.vjp_trajectory(p, states, lam, theta_bar, 0.1, torch.zeros(8, dtype=torch.uint8))
