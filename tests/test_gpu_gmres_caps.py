"""Iteration caps of the outer iterations: a cap far beyond what a run takes (as a caller
writes "no cap") changes nothing."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

NO_CAP = [2**30, 2**31 - 1]


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


def problem(**kw):
    from paper_2404_15249_amd import kfbi
    p = synth.circle_problem(n=64, m=128, kappa=1.0)
    return kfbi.Problem(kfbi.Context(0), p.xy, p.n, p.kappa, **kw), p


@pytest.mark.parametrize("cap", NO_CAP)
def test_no_cap(cap):
    print(f"cap {cap}", flush=True)
    prob, p = problem()
    x = dev(synth.smooth_density(prob.M, 3))
    for run in (lambda c: prob.gmres(x, max_iter=c), lambda c: prob.gmres_neumann(x, max_iter=c),
                lambda c: prob.richardson(x, gamma=0.8, tol=1e-6, max_iter=c), lambda c: prob.bicgstab(x, max_iter=c)):
        want, got = run(300), run(cap)
        assert want[-1] and got[-1] and want[1:-1] == got[1:-1]
        assert torch.equal(want[0], got[0])
    data = dev(p.f_grid), dev(p.f_gamma), dev(p.g)
    want = prob.solve(*data)
    capped, _ = problem(max_iter=cap)
    for got in (capped.solve(*data), capped.solve_neumann(*data)):
        assert got[-1]
    got = capped.solve(*data)
    assert got[3:] == want[3:] and all(torch.equal(a, b) for a, b in zip(got[:3], want[:3]))


@pytest.mark.parametrize("cap", NO_CAP)
def test_no_cap_3d(cap):
    from paper_2404_15249_amd import kfbi
    print(f"3D, cap {cap}", flush=True)
    prob = kfbi.Problem3(kfbi.Context(0), 64, kappa=50.0, tol=1e-6)
    x = dev(synth.smooth_density3(prob.points()[0], 3))
    want, got = prob.gmres(x, tol=1e-6), prob.gmres(x, tol=1e-6, max_iter=cap)
    assert want[-1] and got[-1] and want[1:-1] == got[1:-1] and torch.equal(want[0], got[0])
