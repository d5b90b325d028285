"""A request of a batch whose iteration overflows between the steps (finite data on a box
of 1e-76: the corrections divide by h^2): it alone is stopped, and the others' results
are bitwise what they are without it."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


def overflowing(kfbi, ctx, m):
    s = 1e-76
    t = 2 * np.pi * np.arange(m) / m
    prob = kfbi.Problem(ctx, 0.8 * s * np.stack([np.cos(t), np.sin(t)], 1), 64, 0.0, lo=-1.2 * s, hi=1.2 * s)
    zero = torch.zeros((65, 65), dtype=torch.float64, device="cuda:0")
    return prob, (zero, zero[0, :1].expand(m).contiguous(), dev(5e152 * np.cos(3 * t) / (m / 128) ** 0.5))


def test_the_others_are_left_alone():
    from paper_2404_15249_amd import kfbi
    ctx = kfbi.Context(0)
    probs = [synth.circle_problem(n=64, m=128), synth.star_problem(n=256, kappa=1.0), synth.star_problem(n=512, kappa=2.0)]
    made = [(kfbi.Problem(ctx, p.xy, p.n, p.kappa), (dev(p.f_grid), dev(p.f_gamma), dev(p.g))) for p in probs]
    bad = [overflowing(kfbi, ctx, m) for m in (128, 200, 256)]
    with pytest.raises(kfbi.NonfiniteError):
        bad[0][0].gmres(bad[0][1][2])
    want = None
    for with_bad in (False, True):
        batch = kfbi.Batch(ctx, max_slots=8, m_max=2048)
        order = [made[0], bad[0], made[1], bad[1], made[2], bad[2]] if with_bad else made
        slots = [(batch.admit(prob, *data), (prob, data) in made) for prob, data in order]
        for _ in range(100):
            batch.step(1)
            state, iters, rel = batch.poll()
            if all(state[s] for s, _ in slots):
                break
        got = []
        for s, healthy in slots:
            if healthy:
                got.append((int(state[s]), int(iters[s]), float(rel[s]), [t.clone() for t in batch.finish(s)[:3]]))
                continue
            assert state[s] == -3
            with pytest.raises(kfbi.NonfiniteError):
                batch.finish(s)
        batch.close()
        torch.cuda.synchronize()
        want = want or got
        for a, b in zip(got, want):
            assert a[:3] == b[:3] and a[0] == 1
            assert all(torch.equal(u, v) for u, v in zip(a[3], b[3]))
