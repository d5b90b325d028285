"""A problem admitted to a batch may be used for other calls between the batch's steps:
applies of either operator (also refused ones), the other outer iterations, and the
autotuner.  The batch's result is bitwise what it is without them."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


def refused(prob, x):
    from paper_2404_15249_amd import kfbi
    bad = x.clone()
    bad[3] = float("nan")
    with pytest.raises(kfbi.NonfiniteError):
        prob.apply(bad)


def autotune(prob, x):
    t = prob.tiles()
    prob.autotune(reps=1)
    prob.set_tiles(t["modes_per_group"], t["dst_cols"])


BETWEEN = {
    "apply": lambda prob, x: prob.apply(x),
    "apply_neumann": lambda prob, x: prob.apply_neumann(x),
    "refused": refused,
    "richardson": lambda prob, x: prob.richardson(x, max_iter=3, tol=1e-30),
    "bicgstab": lambda prob, x: prob.bicgstab(x, max_iter=3, tol=1e-30),
    "autotune": autotune,
}


@pytest.mark.parametrize("n", [64, 256])
def test_calls_between_the_steps_leave_the_batch_alone(n):
    from paper_2404_15249_amd import kfbi
    ctx = kfbi.Context(0)
    p = synth.circle_problem(n=64, m=128) if n == 64 else synth.star_problem(n=n, kappa=1.0)
    prob = kfbi.Problem(ctx, p.xy, p.n, p.kappa)
    other = kfbi.Problem(ctx, p.xy, p.n, p.kappa + 2.0)
    x = dev(synth.smooth_density(prob.M, 3))
    f, fg, g = dev(p.f_grid), dev(p.f_gamma), dev(p.g)
    want = None
    for name in (None, *BETWEEN):
        print(f"n={n} between the steps: {name}", flush=True)
        batch = kfbi.Batch(ctx, max_slots=2, m_max=prob.M)
        slot = batch.admit(prob, f, fg, g)
        second = batch.admit(other, f, fg, g)
        for k in range(60):
            if name and k < 4:                              # before the first step too
                BETWEEN[name](prob, x)
            batch.step(2)
            state, iters, rel = batch.poll()
            if state[slot] and state[second]:
                break
        got = [int(state[slot]), int(iters[slot]), float(rel[slot])]
        out = [t.clone() for t in batch.finish(slot)[:3]]
        batch.close()
        torch.cuda.synchronize()
        if name is None:
            want, want_out = got, out
            assert got[0] == 1
        else:
            assert got == want, name
            assert all(torch.equal(a, b) for a, b in zip(out, want_out)), name
