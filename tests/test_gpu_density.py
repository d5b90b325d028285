"""The launch that checks a density and makes its spline and corrections: sample
counts around its workgroups' edges against the oracle (relative 1e-12, as the other
apply tests: FP64 rounding below 1e-13 times a condition below 10), a NaN or Inf at
each of those places, and the calls after a refused one."""
import numpy as np
import pytest
import torch

from oracle import kfbi_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [63, 193, 194, 195, 387, 388, 389])
def test_density_edges(m):
    from paper_2404_15249_amd import kfbi
    t = 2 * np.pi * np.arange(m) / m
    xy = np.stack([0.8 * np.cos(t), 0.8 * np.sin(t)], axis=1)
    prob = kfbi.Problem(kfbi.Context(0), xy, 256, 2.0)
    plan = O.build_plan(xy, 256, -1.2, 1.2)
    values = np.cos(t) + 0.4 * np.sin(5 * t) + 0.1
    want = O.apply_KD(plan, values, 2.0)
    want_n = O.apply_KN(plan, values, 2.0)
    good = torch.as_tensor(values, device="cuda:0")
    out = torch.full((m,), 7.0, dtype=torch.float64, device="cuda:0")
    for at in sorted({0, 30, 193, 194, m - 1} & set(range(m))):
        bad = good.clone()
        bad[at] = float("nan") if at % 2 else float("-inf")
        out.fill_(7.0)
        for call in (prob.apply, prob.apply_neumann):
            with pytest.raises(kfbi.NonfiniteError):
                call(bad, out)
            assert (out == 7.0).all()
        got = prob.apply(good, out).cpu().numpy()
        assert np.abs(got - want).max() < 1e-12 * np.abs(want).max()
        got = prob.apply_neumann(good).cpu().numpy()
        assert np.abs(got - want_n).max() < 1e-12 * np.abs(want_n).max()
