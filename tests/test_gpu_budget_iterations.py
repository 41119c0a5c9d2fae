"""budget_threshold without iterations: the lower end of its range, for a
negative count as for none (range(iters) is empty for both)."""
import pytest
import torch

from paper_2410_21888_amd import screen as SC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("iters", [0, -1, -7])
def test_no_iterations(iters):
    pred = torch.full((3, 3), -5.0, dtype=torch.float64, device="cuda:0")
    assert SC.budget_threshold(pred, 3, 1.0, iters=iters) == -30.0
    assert SC.budget_threshold(pred, 3, 1.0, iters=1) == -15.0
