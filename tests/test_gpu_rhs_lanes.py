"""Right-hand side with one and two panels per lane: panel counts on both sides of
the rule for either precision, with a partly filled last block.

Tolerances as for the other site kernels: sums of a few hundred FP64 terms of mixed
sign stay within 1e-12 of the largest entry, FP32 terms within 2e-5 of it.
"""

import numpy as np
import pytest

from oracle import multipoles as mp
from synth import icosphere, random_multipoles, sites_in_ball

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,level,tol", [
    ("fp64", 5, 1e-12), ("fp64", 6, 1e-12), ("mixed", 6, 2e-5), ("mixed", 7, 2e-5)])
def test_rhs_on_either_side_of_the_lane_rule(precision, level, tol):
    from paper_1810_03698_amd import Solver
    verts, tris = icosphere(level, radius=6.0)
    v2, t2 = icosphere(1, radius=2.0)  # 80 panels: the last block is not full
    tris = np.concatenate([tris, t2 + len(verts)])
    verts = np.concatenate([verts, v2 + [20.0, 0.0, 0.0]])
    rng = np.random.default_rng(level)
    xyz = sites_in_ball(rng, 130, radius=4.0, min_sep=0.2)
    q, d, Q9, alpha = random_multipoles(rng, 130)
    s = Solver(eps_in=1.0, eps_out=80.0, kappa=0.125, mode="direct", precision=precision)
    s.set_mesh(verts, tris)
    s.set_sites(xyz, q, d, Q9, alpha)
    ref = mp.rhs(verts[tris].mean(axis=1), xyz, q, d, Q9, 1.0)
    assert np.abs(s.rhs(d) - ref).max() < tol * np.abs(ref).max()
