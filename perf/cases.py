"""Performance cases of the boundary-integral solver: what a program asks of it.

A case is one kind of call on one surface:

  product   y = A x or A^T x on device tensors (an outer Krylov method, a
            preconditioner study, an adjoint): `Solver.matvec`
  sites     one step of a caller's own induced-dipole loop: `Solver.rhs`, then
            `Solver.site_fields`
  solve     one solvation energy with its surface densities and dipoles
  gradient  a solve and its backward: one force evaluation at fixed geometry
  geometry  a new geometry on a living context: set_mesh, set_sites, solve,
            backward, as one step of an optimisation or of finite differences

Sizes are those of the repository's workloads (icospheres of 1280 to 81920
panels around 8 sites; a ligand with 8k panels, a 1000-atom globule
with 30k, a 5000-atom one with 144k) and everything between them: a sphere of
frequency f has 20 f^2 panels.  Molecular surfaces are star-shaped ones with
an atom-sized bump at every surface atom, at 7 panels per square Angstrom, and
the sites fill the inside at the density of the globules.

The FP64 results are returned as they come.  The mixed-precision far field is
single precision, so a program that asked for it keeps its results as float32.
"""

import functools
import math

import numpy as np
import torch

from paper_1810_03698_amd import Solver

FOUR_PI = 4.0 * math.pi
EPS_IN, EPS_OUT, KAPPA, THOLE = 1.0, 80.0, 0.125, 0.39
PANELS_PER_A2 = 7.0
F64 = torch.float64


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # smallest call: the 1280-panel sphere, where launches and latency count
        _product("product_sphere_1280_mixed", "sphere", 8, "mixed"),
        # an FP64 reference product on a ligand-sized surface (AUTO: direct)
        _product("product_ligand_8k_fp64", "molecule", 20, "fp64"),
        # the largest sizes at which AUTO still sums directly
        _product("product_19k_mixed", "molecule", 31, "mixed"),
        # a 1000-atom globule's surface (treecode, P 4): the default precision,
        # and the adjoint's FP64 transposed product on an odd neighbour of it
        _product("product_30k_mixed", "molecule", 38, "mixed"),
        _product("product_30k_fp64_transposed", "molecule", 39, "fp64", transpose=True),
        # a 5000-atom globule's surface (treecode, P 5), the largest workload
        _product("product_144k_mixed", "molecule", 85, "mixed", order=5),
        _product("product_144k_fp64", "molecule", 85, "fp64", order=5),
        # site kernels at the largest size, in a caller's own dipole loop
        dict(name="sites_144k_mixed", kind="sites", surface="molecule", f=85, sites=5000,
             precision="mixed", order=5, leaf=300, kappa=KAPPA),
        # one energy: the small verification sphere in FP64, a globule in mixed
        _solve("solve_sphere_1280_fp64", "solve", "sphere", 8, 8, "fp64", restart=50),
        _solve("solve_30k_mixed", "solve", "molecule", 38, 1000, "mixed", restart=200),
        # forces: at fixed geometry in FP64, and a whole step at a new geometry
        _solve("gradient_sphere_2k_fp64", "gradient", "sphere", 11, 8, "fp64", restart=50),
        _solve("geometry_ligand_8k_mixed", "geometry", "molecule", 20, 100, "mixed",
               restart=200),
    ]


def _product(name, surface, f, precision, transpose=False, order=4, leaf=300, kappa=KAPPA):
    return dict(name=name, kind="product", surface=surface, f=f, precision=precision,
                transpose=transpose, order=order, leaf=leaf, kappa=kappa)


def _solve(name, kind, surface, f, sites, precision, restart, order=4, leaf=300, kappa=KAPPA):
    return dict(name=name, kind=kind, surface=surface, f=f, sites=sites, precision=precision,
                restart=restart, order=order, leaf=leaf, kappa=kappa)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the whole range, FP64 and the transposed
    product up to 60k panels, whole solves up to the 1000-atom globule."""
    kind = rng.choices(["product", "sites", "solve", "gradient", "geometry"],
                       [10, 3, 3, 2, 2])[0]
    precision = rng.choice(["mixed", "mixed", "fp64"])
    order = rng.choice([4, 4, 5, 6])
    leaf = rng.choice([150, 300, 300, 400])
    kappa = rng.choice([KAPPA, KAPPA, 0.05, 0.25])
    if kind == "product":
        c = _product(None, rng.choice(["molecule", "sphere"]), 0, precision,
                     transpose=rng.random() < 0.3, order=order, leaf=leaf, kappa=kappa)
        top = 64 if c["surface"] == "sphere" else 85
        c["f"] = _log_int(rng, 8, 55 if precision == "fp64" or c["transpose"] else top)
    elif kind == "sites":
        f = _log_int(rng, 10, 85 if precision == "mixed" else 50)
        c = dict(kind=kind, surface="molecule", f=f, sites=_sites_for(f, rng),
                 precision=precision, order=order, leaf=leaf, kappa=kappa)
    else:
        small = kind != "solve" or precision == "fp64"
        if rng.random() < 0.5:
            surface, f, sites = "sphere", _log_int(rng, 8, 16 if small else 40), 8
        else:
            surface, f = "molecule", _log_int(rng, 12, 15 if small else 36)
            sites = _sites_for(f, rng)
        c = _solve(None, kind, surface, f, sites, precision,
                   restart=50 if surface == "sphere" else 200, order=order, leaf=leaf,
                   kappa=kappa)
    c.pop("name", None)
    return c


def _sites_for(f, rng):
    """A site count between a sparse and a full inside of that surface."""
    return max(4, int(0.38 * (_radius(f) - 2.0) ** 3 * rng.uniform(0.4, 1.0)))


# --------------------------------------------------------------------- inputs
def _radius(f):
    """Base radius of a molecular surface with 20 f^2 panels (its bumps add
    about 30 % to the sphere's area)."""
    return math.sqrt(20 * f * f / (PANELS_PER_A2 * FOUR_PI * 1.3))


@functools.lru_cache(maxsize=8)
def _geodesic(f):
    """Unit sphere: the icosahedron's faces cut into f^2 triangles each."""
    g = (1 + 5 ** 0.5) / 2
    v = np.array([(-1, g, 0), (1, g, 0), (-1, -g, 0), (1, -g, 0), (0, -1, g), (0, 1, g),
                  (0, -1, -g), (0, 1, -g), (g, 0, -1), (g, 0, 1), (-g, 0, -1), (-g, 0, 1)])
    v /= np.linalg.norm(v[0])
    faces = np.array([(0, 11, 5), (0, 5, 1), (0, 1, 7), (0, 7, 10), (0, 10, 11), (1, 5, 9),
                      (5, 11, 4), (11, 10, 2), (10, 7, 6), (7, 1, 8), (3, 9, 4), (3, 4, 2),
                      (3, 2, 6), (3, 6, 8), (3, 8, 9), (4, 9, 5), (2, 4, 11), (6, 2, 10),
                      (8, 6, 7), (9, 8, 1)])
    i, j = np.meshgrid(np.arange(f + 1), np.arange(f + 1), indexing="ij")
    keep = i + j <= f
    i, j = i[keep], j[keep]
    w = np.stack([f - i - j, i, j], 1) / f                       # barycentric lattice
    at = np.full((f + 1, f + 1), -1)
    at[i, j] = np.arange(len(i))
    ui, uj = i[i + j < f], j[i + j < f]
    up = np.stack([at[ui, uj], at[ui + 1, uj], at[ui, uj + 1]], 1)
    di, dj = i[i + j < f - 1], j[i + j < f - 1]
    down = np.stack([at[di + 1, dj], at[di + 1, dj + 1], at[di, dj + 1]], 1)
    tri = np.concatenate([up, down])
    pts = np.concatenate([w @ v[t] for t in faces])
    tris = np.concatenate([tri + k * len(w) for k in range(20)])
    _, first, inv = np.unique(np.round(pts * 1e7).astype(np.int64), axis=0,
                              return_index=True, return_inverse=True)
    pts = pts[first]
    pts /= np.linalg.norm(pts, axis=1, keepdims=True)
    return pts, inv.reshape(-1)[tris].astype(np.int32)


def _surface(case, gen):
    """Vertices and triangles on the device, outward orientation."""
    u, tris = _geodesic(case["f"])
    u = torch.as_tensor(u, device="cuda")
    tris = torch.as_tensor(tris, device="cuda")
    if case["surface"] == "sphere":
        # any orientation of the sphere against the sites and the octree
        q, _ = torch.linalg.qr(torch.randn(3, 3, generator=gen, dtype=F64, device="cuda"))
        q = q * torch.sign(torch.det(q))
        return (4.0 * u @ q).contiguous(), tris
    # an atom about every 2.4 A of the surface; its cap above the base sphere,
    # blended over 0.35 A
    radius = _radius(case["f"])
    n = max(12, int(FOUR_PI * radius ** 2 / 5.8))
    at = torch.randn(n, 3, generator=gen, dtype=F64, device="cuda")
    at /= at.norm(dim=1, keepdim=True)
    depth = radius - 1.2 * torch.rand(n, generator=gen, dtype=F64, device="cuda")
    size = 1.2 + 0.8 * torch.rand(n, generator=gen, dtype=F64, device="cuda")
    tau, rows = 0.35, []
    for b in u.split(8192):
        d2 = depth ** 2 * 2.0 * (1.0 - b @ at.T)
        top = torch.clamp(depth + size - d2 / (2.0 * size), min=0.0)
        floor = torch.full((len(b), 1), radius - 0.5, dtype=F64, device="cuda")
        rows.append(tau * torch.logsumexp(torch.cat([top, floor], 1) / tau, 1))
    return (u * torch.cat(rows)[:, None]).contiguous(), tris


def _sites(case, gen):
    """Polarisable multipoles: 8 near the centre of the sphere, else spread
    over the inside of the surface, none closer than 1.2 A to another."""
    m = case["sites"]
    inner = 2.5 if case["surface"] == "sphere" else _radius(case["f"]) - 2.0
    h = inner * (FOUR_PI / 3.0 / (1.3 * m)) ** (1.0 / 3.0)
    k = int(inner / h) + 2
    g = torch.arange(-k, k + 1, dtype=F64, device="cuda") * h
    p = torch.cartesian_prod(g, g, g)
    p = p + min(0.35, 0.2 * h) * (2.0 * torch.rand(p.shape, generator=gen, dtype=F64,
                                                   device="cuda") - 1.0)
    rank = p.norm(dim=1) + 0.3 * h * torch.rand(len(p), generator=gen, dtype=F64,
                                                device="cuda")
    p = p[torch.argsort(rank)[:m]]

    def rand(*shape):
        return torch.rand(*shape, generator=gen, dtype=F64, device="cuda")

    q = rand(m) - 0.5
    d = torch.randn(m, 3, generator=gen, dtype=F64, device="cuda")
    d = d / d.norm(dim=1, keepdim=True) * (0.3 * rand(m, 1))
    Q = 0.2 * torch.randn(m, 3, 3, generator=gen, dtype=F64, device="cuda")
    Q = 0.5 * (Q + Q.transpose(1, 2))
    tr = Q.diagonal(dim1=1, dim2=2).sum(1) / 3.0
    Q = Q - tr[:, None, None] * torch.eye(3, dtype=F64, device="cuda")
    return p.contiguous(), q, d.contiguous(), Q.reshape(m, 9).contiguous(), 0.3 + 1.2 * rand(m)


def _panels(verts, tris):
    v = verts[tris.long()]
    cr = torch.linalg.cross(v[:, 1] - v[:, 0], v[:, 2] - v[:, 0])
    area2 = cr.norm(dim=1)
    return v, v.mean(1), cr / area2[:, None], 0.5 * area2


def _density(verts, tris, gen):
    """A surface density as the Krylov method meets it: the potential of a few
    charges inside and its normal derivative, and a tenth of noise."""
    _, c, n, _ = _panels(verts, tris)
    src = 0.3 * verts.norm(dim=1).min() * torch.randn(12, 3, generator=gen, dtype=F64,
                                                      device="cuda").clamp(-1, 1)
    q = torch.randn(12, generator=gen, dtype=F64, device="cuda")
    R = c[:, None, :] - src[None]
    ri = 1.0 / R.norm(dim=2)
    phi = ri @ q
    dphi = -((R * n[:, None, :]).sum(2) * ri ** 3) @ q
    x = torch.cat([phi / phi.abs().mean(), dphi / dphi.abs().mean()])
    return x + 0.1 * torch.randn(len(x), generator=gen, dtype=F64, device="cuda")


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 + seed)
    verts, tris = _surface(case, gen)
    inp = dict(verts=verts, tris=tris)
    if "sites" in case:
        inp["sites"] = _sites(case, gen)
    if case["kind"] in ("product", "sites"):
        inp["x"] = _density(verts, tris, gen)
    if case["kind"] == "sites":
        inp["p"] = inp["sites"][2] + 0.1 * torch.randn(case["sites"], 3, generator=gen,
                                                       dtype=F64, device="cuda")
    return inp


def prepare(case, seed):
    inp = _inputs(case, seed)
    # the library's work is queued on the program's own stream, with the
    # tensors that it takes and gives
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        s = Solver(eps_in=EPS_IN, eps_out=EPS_OUT, kappa=case["kappa"], mode="auto",
                   theta=0.5, order_P=case["order"], leaf_panels=case["leaf"],
                   gmres_restart=case.get("restart", 50), gmres_tol=1e-8,
                   scf_tol_debye=1e-8, thole_a=THOLE, precision=case["precision"],
                   stream=stream.cuda_stream)
        s.set_mesh(inp["verts"], inp["tris"])
        if "sites" in inp:
            s.set_sites(*inp["sites"])
    return dict(case=case, solver=s, stream=stream, **inp)


# ----------------------------------------------------------------- one pass
def run(state):
    case, s = state["case"], state["solver"]
    single = case["precision"] == "mixed"
    with torch.cuda.stream(state["stream"]):
        if case["kind"] == "product":
            y = s.matvec(state["x"], transpose=case["transpose"])
            return y.float() if single else y
        if case["kind"] == "sites":
            f, r = s.rhs(state["p"]), s.site_fields(state["x"])
            return (f.float(), r.float()) if single else (f, r)
        if case["kind"] == "geometry":
            s.set_mesh(state["verts"], state["tris"])
            s.set_sites(*state["sites"])
        r = s.solve()
        out = {k: r[k] for k in ("dG", "dG_solv", "dG_pol", "G_vac", "phi", "dphidn",
                                 "mu_diss", "mu_vac")}
        if case["kind"] != "solve":
            g = s.backward()
            out.update({"g_" + k: g[k] for k in ("xyz", "q", "d", "Q9", "verts")})
        return {k: np.float32(v) if single else np.float64(v) for k, v in out.items()}


# ------------------------------------------------------------- work of a pass
def _product_flops(case):
    """33 FLOP per (target, far node) pair summed directly; with the treecode,
    11 leaves per target and some 190 expansions of about 4 (P + 2)^2 terms."""
    n = 20 * case["f"] ** 2
    if n <= 20000:
        return 33.0 * 3 * n * n
    return n * (11 * case["leaf"] * 3 * 33.0 + 190 * 4 * 2 * (case["order"] + 2) ** 2)


def work(case):
    n, m, p = 20 * case["f"] ** 2, case.get("sites", 0), _product_flops(case)
    size = 8 if case["precision"] == "fp64" else 4
    rows = 16 * size * n                       # panel records, near corrections aside
    if case["kind"] == "product":
        return dict(bytes=rows + 16 * n + 2 * size * n, flops=p)
    sites = 40.0 * n * m + 160.0 * 3 * n * m   # right-hand side and full readout
    if case["kind"] == "sites":
        return dict(bytes=rows + 16 * n + size * (n + 10 * m) + 80 * m, flops=sites)
    # about 10 dissolved steps of 15 (sphere) or 40 (molecule) Arnoldi steps
    steps = 10 * (15 if case["surface"] == "sphere" else 40)
    out = dict(bytes=steps * (rows + 16 * n), flops=steps * p + 10 * sites)
    if case["kind"] != "solve":
        out = dict(bytes=2 * out["bytes"], flops=2 * out["flops"] + 10 * p)
    return out


# -------------------------------------------- the same in plain 64-bit torch
def _near_rule():
    """Dunavant's symmetric 19-point rule of degree 9."""
    b, w = [[1 / 3, 1 / 3, 1 / 3]], [0.097135796282799]
    for wt, p in ((0.031334700227139, 0.489682519198738), (0.077827541004774, 0.437089591492937),
                  (0.079647738927210, 0.188203535619033), (0.025577675658698, 0.044729513394453)):
        b += [[1 - 2 * p, p, p], [p, 1 - 2 * p, p], [p, p, 1 - 2 * p]]
        w += 3 * [wt]
    p = (0.036838412054736, 0.221962989160766, 0.741198598784498)
    for o in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)):
        b.append([p[k] for k in o])
        w.append(0.043283539377289)
    return (torch.tensor(b, dtype=F64, device="cuda"), torch.tensor(w, dtype=F64, device="cuda"))


_FAR = ((2 / 3, 1 / 6, 1 / 6), (1 / 6, 2 / 3, 1 / 6), (1 / 6, 1 / 6, 2 / 3))


def _distance(a, b):
    return sum((a[:, None, d] - b[None, :, d]) ** 2 for d in range(3)).sqrt_()


def _terms(r, nR, kappa):
    ri = 1.0 / r
    ri3 = ri ** 3
    e = torch.exp(-kappa * r)
    return ri, nR * ri3, e * ri, nR * ri3 * e * (1.0 + kappa * r)


def _self_values(v, c, kappa):
    """V_L and V_Y of a panel at its own centroid, edge by edge."""
    gx, gw = (torch.as_tensor(a, device="cuda") for a in np.polynomial.legendre.leggauss(48))
    lap, yuk = torch.zeros(len(c), dtype=F64, device="cuda"), 0.0
    for e in range(3):
        a, b = v[:, e] - c, v[:, (e + 1) % 3] - c
        t = (b - a) / (b - a).norm(dim=1, keepdim=True)
        h = torch.linalg.cross(a, t).norm(dim=1)
        ua, ub = torch.asinh((a * t).sum(1) / h), torch.asinh((b * t).sum(1) / h)
        lap = lap + h * (ub - ua)
        u = 0.5 * (ua + ub)[:, None] + 0.5 * (ub - ua)[:, None] * gx
        yuk = yuk + 0.5 * (ub - ua) * ((-torch.expm1(-kappa * h[:, None] * torch.cosh(u)) / kappa
                                        / torch.cosh(u)) @ gw)
    return lap / FOUR_PI, yuk / FOUR_PI


def _blocks(inp, kappa, rows):
    """(first row, [V_L, K_L, V_Y, K_Y]) of `rows` collocation points at a time,
    each [rows, panels]: far rule, near-singular and singular panels."""
    v, c, n, A = _panels(inp["verts"], inp["tris"])
    nb, nw = _near_rule()
    sl, sy = _self_values(v, c, kappa)
    flat = (n * v[:, 0]).sum(1)
    for i0 in range(0, len(c), rows):
        ci = c[i0:i0 + rows]
        nR = ci @ n.T - flat
        M = [0.0, 0.0, 0.0, 0.0]
        for b in _FAR:
            y = sum(b[k] * v[:, k] for k in range(3))
            M = [m + t for m, t in zip(M, _terms(_distance(ci, y), nR, kappa))]
        M = [m.mul_(A / (3 * FOUR_PI)) for m in M]
        i, j = torch.nonzero(_distance(ci, c) < 2.0 * A[i0:i0 + rows].sqrt()[:, None], as_tuple=True)
        R = ci[i][:, None, :] - torch.einsum("qk,ekd->eqd", nb, v[j])
        r = R.norm(dim=2)
        own = j == i + i0
        r[own] = 1.0
        fine = _terms(r, (R * n[j][:, None, :]).sum(2), kappa)
        fine = [(t @ nw) * A[j] / FOUR_PI for t in fine]
        zero = torch.zeros_like(sl)
        for m, t, s in zip(M, fine, (sl, zero, sy, zero)):
            m[i, j] = torch.where(own, s[j], t)
        yield i0, M


def _product_exact(inp, case):
    n, x, e = len(inp["tris"]), inp["x"], EPS_IN / EPS_OUT
    rows = max(1, min(n, int(1e8 / n)))
    if case["transpose"]:
        y = torch.cat([0.5 * (x[:n] + x[n:]), torch.zeros_like(x[:n])])
        for i0, (vl, kl, vy, ky) in _blocks(inp, case["kappa"], rows):
            z1, z2 = x[i0:i0 + len(vl)], x[n + i0:n + i0 + len(vl)]
            y[:n] += z1 @ kl - z2 @ ky
            y[n:] += e * (z2 @ vy) - z1 @ vl
        return y
    y = torch.cat([0.5 * x[:n], 0.5 * x[:n]])
    for i0, (vl, kl, vy, ky) in _blocks(inp, case["kappa"], rows):
        y[i0:i0 + len(vl)] += kl @ x[:n] - vl @ x[n:]
        y[n + i0:n + i0 + len(vl)] += e * (vy @ x[n:]) - ky @ x[:n]
    return y


_UPPER = ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))


def _ten(value, grad, hess):
    return torch.cat([value[..., None], grad] + [hess[..., a, b, None] for a, b in _UPPER], -1)


def _fields_exact(inp, x):
    """Reaction potential, gradient and second derivatives at the sites."""
    v, _, n, A = _panels(inp["verts"], inp["tris"])
    N = len(A)
    sv, sk = A / (3 * FOUR_PI) * x[N:], A / (3 * FOUR_PI) * x[:N]
    eye = torch.eye(3, dtype=F64, device="cuda")
    out = []
    for p in inp["sites"][0].split(max(1, int(4e6 / N))):
        acc = 0.0
        for b in _FAR:
            R = p[:, None, :] - sum(b[k] * v[:, k] for k in range(3))[None]
            i2 = 1.0 / (R * R).sum(2)
            i1 = i2.sqrt()
            i3, i5, i7 = i1 * i2, i1 * i2 ** 2, i1 * i2 ** 3
            nR = (n * R).sum(2)
            w3, w5, w7 = (sk * i3), (sk * i5), (sk * nR * i7)
            value = i1 @ sv - (nR * w3).sum(1)
            grad = (-(sv * i3 - 3 * nR * w5)[..., None] * R).sum(1) - w3 @ n
            RR = torch.bmm(((3 * sv * i5 - 15 * w7)[..., None] * R).transpose(1, 2).contiguous(),
                           R.contiguous())
            nRs = torch.bmm((3 * w5[..., None] * n).transpose(1, 2).contiguous(), R.contiguous())
            hess = RR + nRs + nRs.transpose(1, 2) \
                + ((3 * nR * w5).sum(1) - i3 @ sv)[:, None, None] * eye
            acc = acc + _ten(value, grad, hess)
        out.append(FOUR_PI * acc)
    return torch.cat(out)


def _rhs_exact(inp, p):
    xyz, q, _, Q9, _ = inp["sites"]
    _, c, _, _ = _panels(inp["verts"], inp["tris"])
    Q, out = Q9.view(-1, 3, 3), []
    for ci in c.split(max(1, int(2e7 / len(q)))):
        R = ci[:, None, :] - xyz[None]
        ri = 1.0 / R.norm(dim=2)
        QR = torch.bmm(R.transpose(0, 1).contiguous(), Q).transpose(0, 1)
        out.append((q * ri + (p * R).sum(2) * ri ** 3 + 0.5 * (QR * R).sum(2) * ri ** 5).sum(1))
    return torch.cat(out) / (FOUR_PI * EPS_IN)


def _pair(xyz):
    R = xyz[:, None, :] - xyz[None]
    r = R.norm(dim=2) + torch.eye(len(xyz), dtype=F64, device="cuda")
    off = 1.0 - torch.eye(len(xyz), dtype=F64, device="cuda")
    return R, 1.0 / r, off


def _permanent_field(inp):
    xyz, q, d, Q9, _ = inp["sites"]
    R, ri, off = _pair(xyz)
    QR = torch.bmm(R.transpose(0, 1).contiguous(), Q9.view(-1, 3, 3)).transpose(0, 1)
    g = ((-q * ri ** 3 - 3 * (d * R).sum(2) * ri ** 5 - 2.5 * (QR * R).sum(2) * ri ** 7)
         * off)[..., None] * R + (ri ** 3 * off)[..., None] * d + (ri ** 5 * off)[..., None] * QR
    return -g.sum(1) / EPS_IN


def _induced_exact(inp, mu):
    """Damped potential data of the induced dipoles at the other sites."""
    xyz, alpha = inp["sites"][0], inp["sites"][4]
    R, ri, off = _pair(xyz)
    s = THOLE / (ri ** 3 * torch.sqrt(alpha[:, None] * alpha[None]))
    e = torch.exp(-s)
    l3, l5, l7 = (1 - e) * off, (1 - (1 + s) * e) * off, (1 - (1 + s + 0.6 * s * s) * e) * off
    uR = (mu * R).sum(2)
    value = (l3 * uR * ri ** 3).sum(1)
    grad = ((l3 * ri ** 3)[..., None] * mu - (3 * l5 * uR * ri ** 5)[..., None] * R).sum(1)
    w5, w7 = 3 * l5 * ri ** 5, 15 * l7 * uR * ri ** 7
    RR = torch.bmm((w7[..., None] * R).transpose(1, 2).contiguous(), R)
    uRs = torch.bmm((w5[..., None] * mu[None]).transpose(1, 2).contiguous(), R)
    hess = RR - uRs - uRs.transpose(1, 2) \
        - (w5 * uR).sum(1)[:, None, None] * torch.eye(3, dtype=F64, device="cuda")
    return _ten(value, grad, hess) / EPS_IN


def _energy(inp, data):
    _, q, d, Q9, _ = inp["sites"]
    H = data[:, [4, 5, 6, 5, 7, 8, 6, 8, 9]]
    e, na, eps0 = 1.602176634e-19, 6.02214076e23, 8.8541878128e-12
    kcal = e * e * na / (FOUR_PI * eps0 * 1e-10 * 4184.0)
    return 0.5 * kcal * float((q * data[:, 0] + (d * data[:, 1:4]).sum(1)
                               + (Q9 * H).sum(1) / 6.0).sum())


def _solve_exact(inp, case):
    """Dense system, factorised; both dipole loops iterated to the last digit."""
    n, e = len(inp["tris"]), EPS_IN / EPS_OUT
    A = torch.zeros(2 * n, 2 * n, dtype=F64, device="cuda")
    for i0, (vl, kl, vy, ky) in _blocks(inp, case["kappa"], 512):
        k = len(vl)
        A[i0:i0 + k, :n], A[i0:i0 + k, n:] = kl, -vl
        A[n + i0:n + i0 + k, :n], A[n + i0:n + i0 + k, n:] = -ky, e * vy
    A[:n, :n].diagonal().add_(0.5)
    A[n:, :n].diagonal().add_(0.5)
    lu, piv = torch.linalg.lu_factor(A)
    d, alpha = inp["sites"][2], inp["sites"][4]
    perm = _permanent_field(inp)

    def density(mu):
        b = torch.cat([_rhs_exact(inp, d + mu), torch.zeros(n, dtype=F64, device="cuda")])
        return torch.linalg.lu_solve(lu, piv, b[:, None])[:, 0]

    def loop(solvent):
        mu = torch.zeros_like(d)
        for _ in range(200):
            field = perm - _induced_exact(inp, mu)[:, 1:4]
            if solvent:
                field = field - _fields_exact(inp, density(mu))[:, 1:4]
            new = 0.3 * mu + 0.7 * alpha[:, None] * field
            step = float((new - mu).norm() / new.norm())
            mu = new
            if step < 1e-14:
                break
        return mu

    mu_vac, mu_diss = loop(False), loop(True)
    x = density(mu_diss)
    solv = _energy(inp, _fields_exact(inp, x))
    pol = _energy(inp, _induced_exact(inp, mu_diss - mu_vac))
    x = FOUR_PI * x
    out = dict(dG=np.float64(solv + pol), dG_solv=np.float64(solv), dG_pol=np.float64(pol),
               G_vac=None, phi=x[:n], dphidn=x[n:], mu_diss=mu_diss, mu_vac=mu_vac)
    if case["kind"] != "solve":
        out.update({"g_" + k: None for k in ("xyz", "q", "d", "Q9", "verts")})
    return out


def exact(case, seed):
    inp = _inputs(case, seed)
    if case["kind"] == "product":
        return _product_exact(inp, case)
    if case["kind"] == "sites":
        return _rhs_exact(inp, inp["p"]), _fields_exact(inp, inp["x"])
    if len(inp["tris"]) > 4000 or case["sites"] > 64:
        return None   # the dense system, or the loops over it, take too long
    return _solve_exact(inp, case)
