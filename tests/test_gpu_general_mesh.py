"""K x and the residual on sheared boxes: general macros whose rows of A and C
couple all fourteen neighbours (on right-angled macros those off the axes vanish).
Volume and interface rows share a launch below 16 intervals per macro edge and on
meshes of fewer than 2560 volume tiles; the others take two.  Against the oracle's
rows on sampled vertices: a row is a sum of at most 500 products (the oracle's, per
tetrahedron), so both sides stay within 500 roundings, 1e-13, of the sum of their
magnitudes."""
import numpy as np
import pytest

import workloads as W
from oracle.rows import stokes_rows
from test_gpu_lattice import _box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHEAR = np.array([[1.0, 0.25, 0.125], [0.0, 1.0, 0.125], [0.375, 0.0, 1.0]])


def _sample(ext, n, rng):
    """Vertices of the lattice: any, and on the planes of the split of the cells
    and between them."""
    top = np.array(ext) * n
    P = rng.integers(0, top + 1, size=(240, 3))
    c = P // n * n
    P[:40, 1] = np.minimum(c[:40, 1] + P[:40, 0] % n, top[1])   # x' = y'
    P[40:80, 2] = np.minimum(c[40:80, 2] + P[40:80, 1] % n, top[2])
    P[80:120] = c[80:120]
    for a in range(3):
        P[120 + 20 * a:140 + 20 * a, a] = c[120 + 20 * a:140 + 20 * a, a]
    return P


@pytest.mark.parametrize("ext,R,nu_max", [((1, 1, 1), 2, 1.0), ((2, 1, 1), 3, 3.0), ((1, 2, 1), 4, 3.0),
                                          ((1, 1, 2), 5, 1.0), ((1, 1, 1), 6, 1.0), ((6, 3, 2), 4, 3.0)])
def test_rows_of_sheared_boxes(ext, R, nu_max):
    import paper_1511_02134_amd as P
    print(f"[gpu-case] sheared box {ext} R={R} nu={nu_max}", flush=True)
    xyz, tet, nu, tags = _box(ext, nu_max, outflow=True)
    phys = xyz @ SHEAR
    n = 1 << R
    nv = [e * n + 1 for e in ext]
    N = int(np.prod(nv))

    def rows(verts, x, f):
        return stokes_rows(xyz, tet, nu, tags, R, verts, x, f, phys=phys)

    # every neighbour of an interior vertex has a coefficient in A and in C
    mid = np.array([[1, 1, 1]]) * (n // 2)
    for d in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (0, 1, 1), (1, 0, 1), (1, 1, 1)):
        q = mid[0] + d
        e = np.zeros((4, N))
        e[0, q[0] + nv[0] * (q[1] + nv[1] * q[2])] = e[3, q[0] + nv[0] * (q[1] + nv[1] * q[2])] = 1.0
        kx = rows(mid, np.stack([e[0], 0 * e[0], 0 * e[0], 0 * e[0]]), np.zeros((3, N)))[1]
        kp = rows(mid, np.stack([0 * e[3], 0 * e[3], 0 * e[3], e[3]]), np.zeros((3, N)))[1]
        assert kx[0, 0] != 0.0 and kp[3, 0] != 0.0, d

    s = P.Solver(xyz, tet, nu, tags, R, phys=phys)
    g = torch.Generator(device="cuda").manual_seed(R)
    xn = torch.randn(4, N, generator=g, dtype=torch.float64, device="cuda")
    bn = torch.randn(4, N, generator=g, dtype=torch.float64, device="cuda")
    _, dmask = s.node_info()
    bn[:3, torch.tensor(dmask, device="cuda")] = 0.0
    x, b = s.scatter(xn), s.scatter(bn)
    y = s.gather(s.apply(x)).cpu().numpy()
    r, nrm = s.residual(x, b)
    r2, nrm2 = torch.empty_like(r), torch.zeros(1, dtype=torch.float64, device="cuda")
    s.residual_noalloc(x, b, r2, nrm2)
    assert torch.equal(s.scatter(s.gather(r)), s.scatter(s.gather(r2)))
    rn = s.gather(r)
    assert nrm == pytest.approx(float(rn.norm()), rel=1e-12) and float(nrm2) == nrm
    verts = _sample(ext, n, np.random.default_rng(R))
    idx = verts[:, 0] + nv[0] * (verts[:, 1] + nv[1] * verts[:, 2])
    _, kx, dirich, scale = rows(verts, xn.cpu().numpy(), np.zeros((3, N)))
    assert np.array_equal(dirich, dmask[idx])
    bs = bn.cpu().numpy()[:, idx]
    assert np.all(np.abs(y[:, idx] - kx) <= 1e-13 * scale)
    keep = np.stack([~dirich] * 3 + [np.ones_like(dirich)])
    assert np.all(np.abs(rn.cpu().numpy()[:, idx] - (bs - kx) * keep) <= 1e-13 * (scale + np.abs(bs)))
