"""The interface solves' own launches: transforms that read and write the caller's
grid, row solves that add the corrections' sums and make the samples' partial sums.
Every tile shape and every combination of inputs and outputs against the oracle
(values relative 1e-12, as the other interface solve tests; normal derivatives, which
divide grid values by h = 2.4 / n, 1e-12 n), and the rows a solve leaves for the next."""
import numpy as np
import pytest
import torch

import synth
from oracle import kfbi_oracle as O

pytestmark = pytest.mark.gpu

LO, HI = synth.BOX_LO, synth.BOX_HI


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


def relerr(a, b):
    torch.cuda.synchronize()
    return float(np.abs(a.cpu().numpy() - b).max() / max(np.abs(b).max(), 1e-300))


def box_nan(f):
    """The same right-hand side with NaN on the box, where no interior node is."""
    f = f.copy()
    f[0, :] = f[-1, :] = f[:, 0] = f[:, -1] = np.nan
    return f


@pytest.mark.parametrize("n,m", [(64, 65), (128, 131), (256, 255), (512, 1025)])
def test_tiles_and_outputs_match_oracle(n, m):
    from paper_2404_15249_amd import kfbi
    print(f"dense solves n={n} m={m}", flush=True)
    xy = synth.circle_points(m, 0.8)
    prob = kfbi.Problem(kfbi.Context(0), xy, n, 2.0)
    plan = O.build_plan(xy, n, LO, HI)
    rng = np.random.default_rng(n)
    f = np.zeros((n + 1, n + 1))
    f[1:n, 1:n] = rng.standard_normal((n - 1, n - 1))
    y, fg = synth.smooth_density(m, 5), synth.smooth_density(m, 6)
    cases = [(y, f, fg), (y, None, None), (None, f, None), (None, f, fg)]
    zero = np.zeros((n + 1, n + 1))
    want = [O.interface_solve(plan, np.zeros(m) if a is None else a, zero if b is None else b, c, 2.0) for a, b, c in cases]
    want_n = [O.interface_solve_neumann(plan, a, zero if b is None else b, c, 2.0) for a, b, c in cases]
    t0 = prob.tiles()
    for rm, cols in [(t0["modes_per_group"], b) for b in (4, 8, 16, 32, 64)] + [(r, t0["dst_cols"]) for r in (1, 2, 4, 8)]:
        try:
            prob.set_tiles(rm, cols)
        except kfbi.KfbiError:
            continue
        for (a, b, c), (v, z), (vn, zn, dn) in zip(cases, want, want_n):
            args = [None if q is None else dev(q) for q in (a, None if b is None else box_nan(b), c)]
            gv, gz = prob.interface_solve(*args)
            assert relerr(gv, v) < 1e-12 and relerr(gz, z) < 1e-12, (rm, cols)
            gv, gz, gd = prob.interface_solve_neumann(*args)
            assert relerr(gv, vn) < 1e-12 and relerr(gz, zn) < 1e-12, (rm, cols)
            assert relerr(gd, dn) < 1e-12 * n, (rm, cols)


@pytest.mark.parametrize("precision,refine", [("fp64", 0), ("fp32", 0), ("fp32", 1), ("fp32", 3)])
@pytest.mark.parametrize("n", [64, 512, 2048])
def test_fast_solve_in_place(n, precision, refine):
    from paper_2404_15249_amd import kfbi
    prob = kfbi.Problem(kfbi.Context(0), synth.circle_points(n, 0.8), n, 1.0, precision=precision, refine_steps=refine)
    rhs = dev(np.random.default_rng(n).standard_normal((n + 1, n + 1)))
    want = prob.fast_solve(rhs)
    assert not want[0].any() and not want[-1].any() and not want[:, 0].any() and not want[:, -1].any()
    prob.fast_solve(rhs, rhs)
    torch.cuda.synchronize()
    assert torch.equal(rhs, want)


def test_batch_finish_after_another_dense_solve():
    """A finish reuses the admission's transformed f only while nothing replaced it."""
    from paper_2404_15249_amd import kfbi
    ctx = kfbi.Context(0)
    p = synth.star_problem(n=128, kappa=1.0)
    prob = kfbi.Problem(ctx, p.xy, p.n, p.kappa)
    f, fg, g = dev(p.f_grid), dev(p.f_gamma), dev(p.g)
    got = []
    for between in (None, "fast", "interface"):
        batch = kfbi.Batch(ctx, max_slots=2, m_max=p.xy.shape[0])
        slot = batch.admit(prob, f, fg, g)
        batch.step(4)
        if between == "fast":
            prob.fast_solve(torch.ones_like(f))
        if between == "interface":
            prob.interface_solve(torch.ones(prob.M, dtype=torch.float64, device="cuda:0"), torch.ones_like(f))
        for _ in range(50):
            if batch.poll()[0][slot] != 0:
                break
            batch.step(4)
        u, ug, phi, _ = batch.finish(slot)
        torch.cuda.synchronize()
        got.append([t.clone() for t in (u, ug, phi)])
        batch.close()
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
