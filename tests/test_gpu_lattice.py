"""The cycles on the structured lattice against the same cycle composed from the
entry points that work in the per-macro layout (hhg_smooth, hhg_residual,
hhg_restrict, hhg_coarse_solve, hhg_prolong_add, hhg_project).  Sizes: the
smallest smoothed level alone, rows shorter and longer than a wave, one wave
and four waves per workgroup, boxes of several cells in every direction (rows
that are no power of two), one viscosity and one per macro, outflow faces,
both orders, both pressure sweeps, every workgroup order.

Both sides round differently; a cycle is a fixed sequence of about a hundred
sums of at most 60 terms with a contracting error, so two of them stay within
1e-11 of each other in FP64 (1e4 times the FP64 rounding of such a sum); an
FP32 cycle within 1e-4 of its FP64 counterpart (the same factor over the FP32
rounding, of the correction)."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import workloads as W


def _box(ext, nu_max=1.0, outflow=False, seed=3):
    """Kuhn mesh of the box [0,a]x[0,b]x[0,c]; outflow: natural face at x = a."""
    nv = [e + 1 for e in ext]
    xyz = np.array([(x, y, z) for z in range(nv[2]) for y in range(nv[1]) for x in range(nv[0])], float)
    tet = []
    for cz, cy, cx in itertools.product(range(ext[2]), range(ext[1]), range(ext[0])):
        for s in itertools.permutations((0, 1, 2)):
            v = [cx, cy, cz]
            path = []
            for q in range(4):
                path.append(v[0] + nv[0] * (v[1] + nv[1] * v[2]))
                if q < 3:
                    v[s[q]] += 1
            tet.append(path)
    tet = np.array(tet, np.int32)
    tags = W.boundary_face_tags(tet)
    if outflow:
        for t, f in zip(*np.nonzero(tags)):
            if np.all(xyz[np.delete(tet[t], f)][:, 0] == ext[0]):
                tags[t, f] = W.FACE_NATURAL
    rng = np.random.default_rng(seed)
    nu = np.exp(rng.uniform(-np.log(nu_max), np.log(nu_max), len(tet))) if nu_max > 1 else np.ones(len(tet))
    return xyz, tet, nu, tags


def _composed(s, l, top, x, b):
    """x <- one V-cycle from level l, by the per-macro entry points."""
    o = s.opts
    extra = 2 * (top - l) if o.cycle else 0
    s.smooth(x, b, o.nu1 + extra, l)
    r, _ = s.residual(x, b, l, norm=False)
    bc = s.restrict(r, l)
    if l == 1:
        xc, _, _ = s.coarse_solve(bc)
    else:
        xc = s.vector(l - 1)
        _composed(s, l - 1, top, xc, bc)
    s.prolong_add(xc, x, l)
    s.smooth(x, b, o.nu2 + extra, l)


CASES = [
    # extents, R, nu, outflow, options
    ((1, 1, 1), 3, 1.0, False, {}),
    ((1, 1, 1), 3, 5.0, False, {"ordering": 2}),
    ((2, 3, 1), 3, 1.0, True, {"ordering": 2, "p_sweep": 1}),
    ((3, 1, 2), 3, 4.0, True, {"p_sweep": 1, "block_order": 2}),
    ((1, 1, 1), 4, 1.0, True, {"cycle": 1, "nu1": 1, "nu2": 2}),
    ((3, 2, 1), 4, 3.0, False, {"ordering": 2, "cycle": 1, "block_order": 0}),
    ((1, 2, 2), 5, 1.0, False, {"ordering": 2}),
    ((5, 1, 1), 5, 2.0, True, {}),
    ((1, 1, 1), 6, 1.0, False, {"ordering": 2, "p_sweep": 1}),
    ((1, 1, 1), 7, 1.0, False, {"ordering": 2, "nu1": 1, "nu2": 1}),
    ((3, 1, 1), 6, 6.0, True, {"nu1": 1, "nu2": 1}),
    # the smallest levels with blocks of 2 x 2 rows
    ((4, 1, 1), 7, 1.0, True, {"ordering": 2, "p_sweep": 1, "nu1": 2, "nu2": 1}),
    ((1, 4, 1), 7, 1.0, False, {"ordering": 2, "block_order": 2, "nu1": 1, "nu2": 2}),
]


@pytest.mark.parametrize("ext,R,nu_max,outflow,opts", CASES)
def test_lattice_cycle_equals_composed_cycle(ext, R, nu_max, outflow, opts):
    import paper_1511_02134_amd as P
    print(f"[gpu-case] lattice {ext} R={R} nu={nu_max} outflow={outflow} {opts}", flush=True)
    mesh = _box(ext, nu_max, outflow)
    s = P.Solver(*mesh, R, **opts)
    s.check_layout()
    gen = torch.Generator(device="cuda").manual_seed(R)
    xn = torch.randn(4, s.num_nodes(), generator=gen, dtype=torch.float64, device="cuda")
    f = torch.randn(3, s.num_nodes(), generator=gen, dtype=torch.float64, device="cuda")
    b = s.rhs(s.scatter(f))
    x0 = s.scatter(xn)          # inhomogeneous Dirichlet values too
    xa, xb = x0.clone(), x0.clone()
    for _ in range(2):
        s.vcycle(xa, b)
        _composed(s, s.L, s.L, xb, b)
        s.project(xb)
    ga, gb = s.gather(xa), s.gather(xb)
    assert float((ga - gb).abs().max() / gb.abs().max()) <= 1e-11
    # every copy of a vertex agrees, padding untouched
    assert torch.equal(s.scatter(ga), xa)
    # the solve runs the same cycles
    xs = x0.clone()
    info = s.solve(xs, b, rtol=1e-300, max_cycles=2)
    assert float((s.gather(xs) - gb).abs().max() / gb.abs().max()) <= 1e-11
    for k, x in ((0, x0), (2, xb)):
        _, nrm = s.residual(x, b)
        assert info["res_hist"][k] == pytest.approx(nrm, rel=1e-9)
    # FP32 cycles: the correction of one cycle
    m = P.Solver(*mesh, R, precision=1, **opts)
    x1, x2 = x0.clone(), x0.clone()
    s.vcycle(x1, b)
    m.vcycle(x2, b)
    d = s.gather(x1 - x0)
    assert float((s.gather(x2) - s.gather(x1)).abs().max() / d.abs().max()) <= 1e-4


@pytest.mark.parametrize("ordering", [0, 2])
def test_lattice_solve_after_viscosity_change(ordering):
    """One viscosity, then one per macro, on the same context: the records and
    the kind of the launches follow."""
    import paper_1511_02134_amd as P
    mesh = _box((2, 1, 1))
    nu = np.exp(np.random.default_rng(8).uniform(-1, 1, 12))
    s = P.Solver(*mesh, 4, ordering=ordering, graphs=1)
    f = torch.randn(3, s.num_nodes(), dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(1))
    fi = s.scatter(f)
    for v in (np.ones(12), nu, np.full(12, 2.0)):
        s.set_viscosity(v)
        t = P.Solver(mesh[0], mesh[1], v, mesh[3], 4, ordering=ordering)
        xs, xt = s.vector(), t.vector()
        a = s.solve(xs, s.rhs(fi), rtol=1e-8)
        c = t.solve(xt, t.rhs(fi), rtol=1e-8)
        assert a["res_hist"] == c["res_hist"] and torch.equal(xs, xt)


@pytest.mark.parametrize("ext,R,nu_max,outflow", [((1, 1, 1), 3, 1.0, False), ((1, 1, 1), 5, 1.0, True),
                                                  ((3, 1, 2), 4, 4.0, False), ((1, 1, 1), 6, 3.0, False)])
def test_lattice_pminres_is_minres(ext, R, nu_max, outflow):
    """Preconditioned MINRES on the lattice: the first iterates minimise the
    residual norm of the preconditioner over the Krylov space spanned with
    hhg_apply and hhg_vel_cycle (per-macro layout).  The minimisation in double
    loses the square of the basis' condition, so the iterates agree to 1e-7."""
    import paper_1511_02134_amd as P
    print(f"[gpu-case] lattice pminres {ext} R={R}", flush=True)
    mesh = _box(ext, nu_max, outflow)
    s = P.Solver(*mesh, R, krylov=1)
    gen = torch.Generator(device="cuda").manual_seed(R)
    f = torch.randn(3, s.num_nodes(), generator=gen, dtype=torch.float64, device="cuda")
    b = s.rhs(s.scatter(f))
    x0 = s.scatter(torch.randn(4, s.num_nodes(), generator=gen, dtype=torch.float64, device="cuda"))
    _, dmask = s.node_info()
    free = torch.ones(4, s.num_nodes(), dtype=torch.float64, device="cuda")
    free[:3, torch.tensor(dmask, device="cuda")] = 0.0
    ijk, _ = s.node_info()
    # lumped pressure mass over 1/nu: sum over the tetrahedra around a vertex of |T| / (4 nu_T)
    pm = torch.zeros(s.num_nodes(), dtype=torch.float64)
    n = 1 << R
    lat = [e * n + 1 for e in ext]
    for t in range(len(mesh[1])):
        v0 = mesh[0][mesh[1][t][0]].astype(int) * n
        ax = [int(np.argmax(mesh[0][mesh[1][t][q + 1]] - mesh[0][mesh[1][t][q]])) for q in range(3)]
        c = np.stack(np.meshgrid(*[np.arange(n)] * 3, indexing="ij"), -1).reshape(-1, 3)
        for s6 in itertools.permutations(range(3)):
            path = [np.zeros(3, int)]
            for q in s6:
                path.append(path[-1] + np.eye(3, dtype=int)[q])
            cen = c + sum(path) / 4
            inside = (cen[:, ax[0]] > cen[:, ax[1]]) & (cen[:, ax[1]] > cen[:, ax[2]])
            for p in path:
                X = v0 + c[inside] + p
                pm.index_add_(0, torch.from_numpy(X[:, 0] + lat[0] * (X[:, 1] + lat[1] * X[:, 2])),
                              torch.full((len(X),), (1 / n) ** 3 / 24 / mesh[2][t], dtype=torch.float64))
    pm = pm.to("cuda")

    def K(v):
        return s.gather(s.apply(s.scatter(v)))

    def prec(v):
        z = s.vector()
        s.vel_cycle(z, s.scatter(v))
        z = s.gather(z)
        z[3] = v[3] / pm
        return z

    r, nrm = s.residual(x0, b)
    v = s.gather(r)
    zs = [prec(v)]
    its = 3
    for _ in range(its - 1):
        q = prec(K(zs[-1]))
        for z in zs:
            q = q - (q * z).sum() / (z * z).sum() * z
        zs.append(q)
    zs = [z / z.norm() for z in zs]
    # min |v - sum y_i K z_i| in the norm of the preconditioner
    A = [K(z) for z in zs]
    PA = [prec(a) for a in A]
    G = torch.stack([torch.stack([(a * p).sum() for p in PA]) for a in A])
    h = torch.stack([(v * p).sum() for p in PA])
    y = torch.linalg.solve(0.5 * (G + G.T), h)
    ref = s.gather(x0) + sum(c * z for c, z in zip(y, zs))
    xs = x0.clone()
    info = s.pminres(xs, b, rtol=0.0, maxit=its)
    got = s.gather(xs)
    if not outflow:
        ref[3] -= (torch.tensor(s.mass_weights(), device="cuda") * ref[3]).sum() / float(np.prod(ext))
    d = s.gather(x0)
    assert info["r0"] == pytest.approx(nrm, rel=1e-12)
    assert float((got - ref).abs().max() / (ref - d).abs().max()) <= 1e-7
    _, end = s.residual(xs, b)
    assert info["r_final"] == pytest.approx(end, rel=1e-9)
