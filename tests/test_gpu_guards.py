"""Products where a guard of the pair terms decides: sheets in contact whose far
nodes fall on other panels' centroids, and screening so strong that
e^{-kappa r} vanishes.

Tolerances: as for the kernel edges, 1e-12 (FP64) and 2e-5 (FP32 far field) of
the largest entry; A and A^T of one set of rounded pair terms agree to 1e-13
and 1e-6 of |z| |x|.
"""

import numpy as np
import pytest

from oracle import bie
from synth import icosphere

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 2e-5}
TOL_T = {"fp64": 1e-13, "mixed": 1e-6}


def _solver(verts, tris, **kw):
    from paper_1810_03698_amd import Solver
    args = dict(eps_in=1.0, eps_out=80.0, kappa=0.125, mode="direct", precision="fp64")
    args.update(kw)
    s = Solver(**args)
    s.set_mesh(verts, tris)
    return s


def _worst(got, ref):
    return np.abs(got - ref).max() / np.abs(ref).max()


# A tetrahedron and another on top of the same face.  The second one's face is
# cut at the midpoints of two edges: a corner triangle, whose centroid is the
# first one's far node (2/3, 1/6, 1/6), and two more, whose centroids are nobody's
# node in either rule.
_FACE = np.array([[0.0, 0.0, 0.0], [4.0, 0.0, 0.0], [1.0, 3.5, 0.0]])


def _touching(corners, below, above):
    v0, v1, v2 = corners
    m1, m2 = 0.5 * (v0 + v1), 0.5 * (v0 + v2)
    verts = np.array([v0, v1, v2, below, v0, v1, v2, m1, m2, above])
    tris = np.array([[0, 1, 2], [1, 0, 3], [2, 1, 3], [0, 2, 3],
                     [4, 8, 7], [7, 8, 6], [7, 6, 5],
                     [4, 7, 9], [7, 5, 9], [5, 6, 9], [6, 8, 9], [8, 4, 9]], dtype=np.int32)
    return verts, tris


def _touching_mesh(kind):
    """Dyadic coordinates, in which node and centroid may agree to the bit, or the
    same turned and shifted, in which they differ by rounding."""
    verts, tris = _touching(_FACE, np.array([1.5, 1.0, -3.0]), np.array([1.75, 1.25, 3.0]))
    if kind == "turned":
        q, _ = np.linalg.qr(np.random.default_rng(12).normal(size=(3, 3)))
        q *= np.sign(np.linalg.det(q))
        verts = verts @ q.T + np.array([0.7, -1.3, 2.1])
    return verts, tris


@pytest.mark.parametrize("mode", ["direct", "treecode"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", ["dyadic", "turned"])
def test_products_on_sheets_in_contact(kind, precision, mode):
    verts, tris = _touching_mesh(kind)
    m = bie.Mesh(verts, tris, 0.125)
    node = (m.verts[tris[0]] * [[2 / 3], [1 / 6], [1 / 6]]).sum(0)
    assert np.linalg.norm(m.cen - node, axis=1).min() < 1e-14
    A = bie.dense_system(m, 1.0, 80.0)
    # all pairs directly in treecode mode too
    s = _solver(verts, tris, precision=precision, mode=mode, theta=0.05, leaf_panels=8)
    rng = np.random.default_rng(2)
    x, z = rng.normal(size=2 * m.N), rng.normal(size=2 * m.N)
    assert _worst(s.matvec(x), A @ x) < TOL[precision]
    assert _worst(s.matvec(z, transpose=True), A.T @ z) < TOL[precision]


@pytest.mark.parametrize("mode", ["direct", "treecode"])
@pytest.mark.parametrize("kind", ["dyadic", "turned"])
def test_vertex_gradient_on_sheets_in_contact(kind, mode):
    """Along an affine map of the whole mesh, which keeps the sheets in contact and
    nodes on centroids, against a central difference: solves at 1e-13 leave it an
    error of 1e-12 |dG| / h = 3e-7 (the third derivative's h^2 / 6 is below
    1e-8), so 2e-6 of the derivative, which is above 1.  And the sum of all
    gradients along a common shift, which is zero."""
    verts, tris = _touching_mesh(kind)
    rng = np.random.default_rng(5)
    centre = verts[:4].mean(axis=0)  # of the first tetrahedron, 0.6 A from its faces
    xyz = centre + 0.15 * rng.normal(size=(2, 3))
    sites = (xyz, np.array([0.4, -0.1]), 0.1 * rng.normal(size=(2, 3)), np.zeros((2, 9)),
             np.array([0.05, 0.08]))
    B = rng.normal(size=(3, 3))
    u = (verts - centre) @ B.T
    u /= np.linalg.norm(u)
    h = 2e-4

    def solved(v):
        s = _solver(v, tris, mode=mode, theta=0.05, leaf_panels=8, gmres_tol=1e-13,
                    scf_tol_debye=1e-12, scf_maxit=500)
        s.set_sites(*sites)
        return s, s.solve(outputs=False)["dG"]

    s, _ = solved(verts)
    back = s.backward(1.0)
    g = back["verts"]
    fd = (solved(verts + h * u)[1] - solved(verts - h * u)[1]) / (2 * h)
    assert abs(fd) > 1.0 and abs(fd - (g * u).sum()) < 2e-6 * abs(fd)
    # 1e-13 of a few hundred pair terms of up to some 1e3
    assert np.abs(g.sum(axis=0) + back["xyz"].sum(axis=0)).max() < 1e-8


@pytest.mark.parametrize("order", [4, 6])
@pytest.mark.parametrize("kappa", [0.0, 40.0, 1e7, 1e30])
def test_tree_product_screening_range(kappa, order):
    """kappa^order beyond the FP32 range, times e^{-kappa r} = 0."""
    from oracle import treecode
    verts, tris = icosphere(4, radius=4.0)
    rng = np.random.default_rng(order)
    verts = verts + rng.normal(scale=1e-4, size=verts.shape)
    m = bie.Mesh(verts, tris, kappa)
    x, z = rng.normal(size=2 * m.N), rng.normal(size=2 * m.N)
    rows = np.sort(rng.choice(m.N, 96, replace=False))
    ref = treecode.Treecode(m, 0.6, order, 40).matvec(x, 1.0, 80.0, rows=rows)
    for precision in ("fp64", "mixed"):
        s = _solver(verts, tris, mode="treecode", theta=0.6, order_P=order, leaf_panels=40,
                    precision=precision, kappa=kappa)
        y, yt = s.matvec(x), s.matvec(z, transpose=True)
        assert _worst(np.concatenate([y[:m.N][rows], y[m.N:][rows]]), ref) < TOL[precision]
        off = abs(z @ y - yt @ x) / (np.linalg.norm(z) * np.linalg.norm(x))
        assert off < TOL_T[precision]
