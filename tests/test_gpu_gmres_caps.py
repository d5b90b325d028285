"""Iteration caps of the outer iterations: a cap far beyond what a run takes (as a caller
writes "no cap") changes nothing, and a run whose tolerance its own rounding keeps out of
reach ends at its cap, with the iterate written, however short its cycles are.  (Started
at a nearly exact guess, the estimate of each cycle passes the tolerance after a step or
two while the true residual stays: every cycle then costs slots of its own.)"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

NO_CAP = [2**30, 2**31 - 1]


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


def problem(kappa=1.0, **kw):
    from paper_2404_15249_amd import kfbi
    p = synth.circle_problem(n=64, m=128, kappa=kappa)
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


def stagnating(gmres, rhs, exact, cap):
    """gmres from guesses a little off the solution."""
    off = dev(np.random.default_rng(1).standard_normal(rhs.numel()))
    for size, tol in ((0.0, 1e-10), (5e-9, 1e-10), (5e-7, 1e-10), (5e-9, 1e-8), (5e-9, 1e-30), (5e-7, 1e-9), (5e-7, 2e-9)):
        guess = exact + size * off
        phi, iters, applies, rel, ok = gmres(rhs, guess, tol=tol, max_iter=cap)
        print(f"guess {size:.0e} off, tol {tol:.0e}: {iters} steps, {applies} applies, rel {rel:.1e}", flush=True)
        if ok:                                              # rounding happened to allow it
            assert rel < tol
            continue
        assert iters == cap
        assert torch.isfinite(phi).all() and float((phi - exact).abs().max()) < 1e-6 * float(exact.abs().max())


@pytest.mark.parametrize("restart,cap", [(50, 500), (50, 60), (1, 40), (2, 41), (3, 1)])
@pytest.mark.parametrize("kappa,eta", [(1.0, 1e-3), (1.0, 1.0), (0.0, 1e-3), (0.0, 1.0)])
def test_a_stagnating_run_ends_at_its_cap(restart, cap, kappa, eta):
    """On the circle at kappa = 0 the double layer is of rank one: cycles of one step."""
    print(f"restart {restart}, cap {cap}, kappa {kappa}, eta {eta}", flush=True)
    prob, _ = problem(kappa, restart=restart)
    full, _ = problem(kappa)
    prob.set_reorth(eta)
    rhs = dev(synth.smooth_density(prob.M, 3))
    stagnating(prob.gmres, rhs, full.gmres(rhs, tol=1e-11)[0], cap)
    if kappa > 0:
        stagnating(prob.gmres_neumann, rhs, full.gmres_neumann(rhs, tol=1e-11)[0], cap)


def test_a_stagnating_run_ends_at_its_cap_3d():
    from paper_2404_15249_amd import kfbi
    prob = kfbi.Problem3(kfbi.Context(0), 64, kappa=50.0)
    exact = dev(synth.smooth_density3(prob.points()[0], 3))
    stagnating(prob.gmres, prob.apply(exact), exact, 300)


def test_a_warm_started_solve_past_its_tolerance():
    """The Dirichlet solve from its own solution: the cap, and the solution written."""
    prob, p = problem(tol=1e-10)
    data = dev(p.f_grid), dev(p.f_gamma), dev(p.g)
    u, ug, phi, _, _, ok = prob.solve(*data)
    assert ok
    again = prob.solve(*data, phi0=phi)
    print(f"from its own solution: {again[3]} steps, converged {again[5]}", flush=True)
    assert again[5] or again[3] == 500
    for a, b in zip(again[:3], (u, ug, phi)):
        assert float((a - b).abs().max()) < 1e-8 * float(b.abs().max())
