"""A context given up before the objects made in it (a garbage collector finalises a
cycle in any order): they stay usable and can be destroyed afterwards."""
import gc

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


def test_objects_outlive_their_context():
    from paper_2404_15249_amd import kfbi
    p = synth.circle_problem(n=64, m=128, kappa=1.0)
    ctx = kfbi.Context(0)
    prob = kfbi.Problem(ctx, p.xy, p.n, p.kappa)
    prob3 = kfbi.Problem3(ctx, 64)
    batch = kfbi.Batch(ctx, max_slots=1, m_max=128)
    gs = kfbi.GrayScott(ctx, synth.gray_scott_samples(64), 64, 0.01)
    x = dev(synth.smooth_density(prob.M, 3))
    want = prob.apply(x)
    ctx.close()
    assert torch.equal(prob.apply(x), want)
    batch.close()
    prob.close()
    prob3.close()
    gs.close()
    torch.cuda.synchronize()


def test_a_cycle_of_objects_is_collected():
    from paper_2404_15249_amd import kfbi
    p = synth.circle_problem(n=64, m=128, kappa=1.0)
    for first in (True, False):
        ctx = kfbi.Context(0)
        prob = kfbi.Problem(ctx, p.xy, p.n, p.kappa)
        cycle = [ctx, prob] if first else [prob, ctx]
        cycle.append(cycle)
        ctx.held = prob.held = cycle
        del ctx, prob, cycle
        gc.collect()
