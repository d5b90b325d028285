"""The autotuner's grid solve is the one that solves make: it leaves a column tile alone
that no launch reads, returns a valid one where they do, and its time is that of a solve."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def make(n, precision="fp64"):
    from paper_2404_15249_amd import kfbi
    return kfbi.Problem(kfbi.Context(0), synth.circle_points(n, 0.8), n, 1.0, precision=precision)


@pytest.mark.parametrize("n,tiles", [(64, (8, 16, 64)), (256, (4, 16, 64)), (512, (8, 32))])
def test_a_tile_that_is_not_read_stays(n, tiles):
    for cols in tiles:
        prob = make(n)
        prob.set_tiles(prob.tiles()["modes_per_group"], cols)
        for _ in range(3):
            t = prob.autotune(reps=2)
            print(f"n={n} tile {cols}: {t}", flush=True)
            assert t["dst_cols"] == cols and t["grid_solve_us"] > 0 and t["apply_us"] > 0


@pytest.mark.parametrize("n,precision", [(1024, "fp64"), (2048, "fp64"), (256, "fp32"), (1024, "fp32")])
def test_a_tile_that_is_read_is_chosen(n, precision):
    prob = make(n, precision)
    rhs = torch.as_tensor(np.random.default_rng(n).standard_normal((n + 1, n + 1)), device="cuda:0")
    want = prob.fast_solve(rhs)
    t = prob.autotune(reps=2)
    print(f"n={n} {precision}: {t}", flush=True)
    assert t["dst_cols"] in (4, 8, 16) and t["grid_solve_us"] > 0
    got = prob.fast_solve(rhs)
    torch.cuda.synchronize()
    # FP32: two solves of 6e-8 times a growth below 1e2 each
    tol = 1e-12 if precision == "fp64" else 1e-9
    assert float((got - want).abs().max()) < tol * float(want.abs().max())
