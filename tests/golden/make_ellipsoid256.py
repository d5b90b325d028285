"""Writes ellipsoid256_oracle.npz: the FP64 oracle on the 256^3 grid of the ellipsoid
(semi-axes 0.9, 0.7, 0.5 in [-1.2, 1.2]^3, kappa = 1.5, every grid-edge crossing a control
point), whose plan takes minutes on the host and so is stored rather than recomputed
inside a GPU test.

Calls only oracle/ (and the seeded input generators in synth/).  Stored, at seeded samples
of 6000 control points and 6000 grid nodes: K_D of a smooth density, and one interface
solve with that density, a right-hand side and its trace.  Regenerate with
``python tests/golden/make_ellipsoid256.py``.
"""
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
sys.path.insert(0, ROOT)

import synth  # noqa: E402
from oracle import kfbi_oracle3d as O3  # noqa: E402

N = 256
AXES = (0.9, 0.7, 0.5)
KAPPA = 1.5
SAMPLE = 6000
SEED = 256


def main():
    op = O3.build_plan(N, synth.BOX_LO, synth.BOX_HI, AXES)
    pr = synth.ellipsoid_problem(n=N, axes=AXES, kappa=KAPPA)
    phi = synth.smooth_density3(op.q_pos, 77)
    fg, _ = pr.boundary_data(op.q_pos)
    rng = np.random.default_rng(SEED)
    point = np.sort(rng.choice(op.M, size=SAMPLE, replace=False))
    node = np.sort(rng.choice((N + 1) ** 3, size=SAMPLE, replace=False))
    applied = O3.apply_KD(op, phi, KAPPA)
    v, vz = O3.interface_solve(op, phi, O3.zero_extension(op, pr.f_grid), fg, KAPPA)
    out = os.path.join(os.path.dirname(os.path.abspath(__file__)), "ellipsoid256_oracle.npz")
    np.savez_compressed(out, n=N, axes=np.asarray(AXES), kappa=KAPPA, M=op.M, irregular=len(op.irr), point=point, node=node,
                        position=op.q_pos[point], applied=applied[point], vz=vz[point], v=v.ravel()[node],
                        scale=np.array([np.abs(applied).max(), np.abs(vz).max(), np.abs(v).max()]))
    print(f"wrote {out}: {op.M} control points")


if __name__ == "__main__":
    main()
