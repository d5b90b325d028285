"""The sparse fast solve's mirrored mode pairs at the edges of its tables: long
column halves cut into pieces (a domain with straight vertical sides), more samples
than threads, few and odd samples, every grid size and every modes-per-workgroup
value, against the oracle.

Tolerance: both solve the same discrete system in FP64; the relative rounding is
below 1e-13 of the largest value times the condition of the spline and the stencil
weights (below 10 here), so 1e-12 (normal derivative: the weights hold 1/h against
values of order one, so times n / 256 above 256).  The library's dense path is no
reference for the normal derivative: its transforms' running sums put its values
1e-11 off at 2048^2, a hundred times as far as the sparse path's.
"""
import numpy as np
import pytest
import torch

from oracle import kfbi_oracle as O

pytestmark = pytest.mark.gpu


def rounded_box(m, half=0.7003, r=0.25):
    """m points, equally spaced, on a square with rounded corners (counter-clockwise)."""
    side = 2 * (half - r)
    per = 4 * side + 2 * np.pi * r
    pts = []
    for s in per * np.arange(m) / m:
        q, s = divmod(s + side / 2, side + np.pi * r / 2)
        q = int(q) % 4
        if s <= side:
            p = np.array([half, s - side / 2])
        else:
            a = (s - side) / r
            p = np.array([half - r + r * np.cos(a), side / 2 + r * np.sin(a)])
        c, d = [(1, 0), (0, 1), (-1, 0), (0, -1)][q]
        pts.append([c * p[0] - d * p[1], d * p[0] + c * p[1]])
    return np.array(pts)


def circle(m, r=0.8):
    t = 2 * np.pi * np.arange(m) / m
    return np.stack([r * np.cos(t), r * np.sin(t)], axis=1)


CASES = [(64, circle(37)), (64, rounded_box(64)), (128, rounded_box(97)), (256, rounded_box(201)),
         (512, rounded_box(1031)), (1024, rounded_box(2050)), (2048, rounded_box(1023)), (2048, circle(2049)),
         (4096, rounded_box(1500))]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_pairs_match_dense(case):
    from paper_2404_15249_amd import kfbi
    n, xy = CASES[case]
    ctx = kfbi.Context(0)
    prob = kfbi.Problem(ctx, xy, n, 1.5)
    m = len(xy)
    t = 2 * np.pi * np.arange(m) / m
    values = 1.0 + np.cos(t) + 0.3 * np.sin(3 * t)
    phi = torch.as_tensor(values, device="cuda:0")
    plan = O.build_plan(xy, n, -1.2, 1.2)
    want = torch.as_tensor(O.apply_KD(plan, values, 1.5), device="cuda:0")
    want_n = torch.as_tensor(O.apply_KN(plan, values, 1.5), device="cuda:0")
    default = prob.tiles()
    tried = 0
    for modes in (1, 2, 4, 8):
        try:
            prob.set_tiles(modes, default["dst_cols"])
        except kfbi.KfbiError:
            continue
        tried += 1
        err = (prob.apply(phi) - want).abs().max() / want.abs().max()
        err_n = (prob.apply_neumann(phi) - want_n).abs().max() / want_n.abs().max()
        print(f"n={n} m={m} modes={modes}: {err:.2e} {err_n:.2e}")
        assert err < 1e-12
        assert err_n < 1e-12 * max(1.0, n / 256)
    assert tried >= 2
