"""Calls that wait for their own work, from a stream that is busy with their input,
from an idle one, and after a call that raised: the same bits each time, and what the
caller enqueues next sees the result."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [False, True])
def test_busy_and_idle_callers(side):
    from paper_2404_15249_amd import kfbi
    ctx = kfbi.Context(0)
    prob = kfbi.Problem(ctx, synth.circle_points(256, 0.8), 128, 1.0)
    phi = torch.as_tensor(synth.smooth_density(prob.M, 3), device="cuda:0")
    torch.cuda.synchronize()
    calls = {"apply": lambda x: prob.apply(x), "neumann": lambda x: prob.apply_neumann(x),
             "gmres": lambda x: prob.gmres(x)[0], "bicgstab": lambda x: prob.bicgstab(x)[0]}
    want = {k: f(phi).clone() for k, f in calls.items()}
    torch.cuda.synchronize()
    stream = torch.cuda.Stream() if side else torch.cuda.current_stream()
    big = torch.ones(4096, 4096, device="cuda:0")
    bad = phi.clone()
    bad[5] = float("nan")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for name, call in calls.items():
            for busy in (True, False):
                x = torch.full_like(phi, float("inf"))
                if busy:
                    for _ in range(4):                       # some milliseconds before x is written
                        big = big @ big
                        big.fill_(1e-3)
                else:
                    stream.synchronize()
                x.copy_(phi)
                if not busy:
                    stream.synchronize()
                got = call(x)
                x.fill_(float("inf"))                        # the call has read x
                assert torch.equal(got, want[name]), (name, busy)
                with pytest.raises(kfbi.NonfiniteError):
                    prob.apply(bad)
