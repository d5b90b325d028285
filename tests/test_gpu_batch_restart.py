"""Batched GMRES with short cycles and forced second Gram-Schmidt passes (slots whose apply
is not used, and so left out) against the single solves.  Both solve to a relative residual
of 1e-10 on operators of condition below 50, so their solutions agree to 1e-8; the partial
sums are grouped differently, so a step count may move by one."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


@pytest.mark.parametrize("restart", [1, 2, 3, 50])
@pytest.mark.parametrize("eta", [0.0, 1e-3, 1.0])
def test_batch_equals_single_solves(restart, eta):
    from paper_2404_15249_amd import kfbi
    ctx = kfbi.Context(0)
    problems = [synth.circle_problem(n=64, m=128, kappa=1.0), synth.star_problem(n=256, kappa=1.0),
                synth.circle_problem(n=128, m=200, kappa=3.0)]
    batch = kfbi.Batch(ctx, max_slots=4, m_max=1024)
    want, slots = [], []
    for p in problems:
        prob = kfbi.Problem(ctx, p.xy, p.n, p.kappa, restart=restart, max_iter=300)
        prob.set_reorth(eta)
        data = dev(p.f_grid), dev(p.f_gamma), dev(p.g)
        want.append(prob.solve(*data))
        slots.append(batch.admit(prob, *data))
    for _ in range(300):
        batch.step(4)
        state, iters, rel = batch.poll()
        if all(state[s] for s in slots):
            break
    for s, w, p in zip(slots, want, problems):
        print(f"{p.name} restart={restart} eta={eta}: {iters[s]} steps, single {w[3]}", flush=True)
        assert w[5] and state[s] == 1 and abs(int(iters[s]) - w[3]) <= 1
        for a, b in zip(batch.finish(s)[:3], w):
            torch.cuda.synchronize()
            assert float((a - b).abs().max()) < 1e-8 * float(b.abs().max())
