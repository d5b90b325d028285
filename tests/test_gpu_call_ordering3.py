"""What the caller enqueues after a three-dimensional apply sees its result."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_apply3_result_is_ordered_before_the_callers_next_work():
    from paper_2404_15249_amd import kfbi
    prob = kfbi.Problem3(kfbi.Context(0), 64, (0.8, 0.7, 0.6))
    phi = torch.as_tensor(np.cos(np.arange(prob.M)), device="cuda:0")
    want = prob.apply(phi)
    torch.cuda.synchronize()
    out = torch.empty_like(phi)
    for _ in range(20):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        prob.apply(phi, out)
        assert torch.equal(out.clone(), want)
