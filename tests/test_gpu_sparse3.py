"""The three-dimensional apply's own solve (half planes in LDS, the stencils' nodes
alone) against the transforms of the whole grid that an interface solve makes: thin,
small and nearly box-wide ellipsoids, centred in the box or not (off the centre a node's
mirror images in y and z are no nodes of the surface), relative 1e-12 of the largest
value as the comparisons with the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [((0.9, 0.7, 0.5), -1.2, 1.2), ((0.4, 1.0, 0.7), -1.2, 1.2), ((1.0, 0.4, 0.4), -1.3, 1.1),
          ((0.6, 0.6, 0.6), -1.0, 1.7), ((0.5, 0.8, 1.0), -1.7, 1.15)]


@pytest.mark.parametrize("kappa", [0.0, 30.0])
@pytest.mark.parametrize("shape", range(len(SHAPES)))
@pytest.mark.parametrize("n", [64, 128])
def test_apply_equals_the_whole_grids_solve(n, shape, kappa):
    from paper_2404_15249_amd import kfbi
    axes, lo, hi = SHAPES[shape]
    print(f"apply n={n} axes={axes} box=[{lo}, {hi}] kappa={kappa}", flush=True)
    prob = kfbi.Problem3(kfbi.Context(0), n, axes, kappa, lo=lo, hi=hi)
    t = np.arange(prob.M)
    phi = torch.as_tensor(np.cos(0.01 * t) + 0.3 * np.sin(1.7 * t), device="cuda:0")
    _, want = prob.interface_solve(phi)
    got = prob.apply(phi)
    torch.cuda.synchronize()
    assert float((got - want).abs().max()) < 1e-12 * float(want.abs().max())
    bad = phi.clone()
    bad[-1] = float("nan")
    out = torch.full_like(phi, 7.0)
    with pytest.raises(kfbi.NonfiniteError):
        prob.apply(bad, out)
    assert (out == 7.0).all()
    assert torch.equal(prob.apply(phi, out), got)
