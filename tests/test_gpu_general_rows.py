"""K x and the residual of general meshes (15-tap rows, a vertex per lane; one
launch below 16 intervals per macro edge, two from there on) against the Kuhn
kernels: the unit cube given with its own corner coordinates as physical ones is
the same operator through the general path.  A row sums at most 105 products, so
the two agree to 105^2 roundings of the largest row: 1.2e-12."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 105 ** 2 * 2.0 ** -53


@pytest.mark.parametrize("R", [2, 3, 4, 5, 6])
def test_general_rows_equal_kuhn_rows(R):
    import paper_1511_02134_amd as P
    print(f"[gpu-case] general rows R={R}", flush=True)
    xyz, tet = W.box_mesh(1)
    tags = W.face_tags(xyz, tet, 1, None)
    mesh = (xyz, tet, np.linspace(0.5, 2.0, tet.shape[0]), tags)
    k = P.Solver(*mesh, R)
    g = P.Solver(*mesh, R, phys=np.asarray(xyz, float))
    gen = torch.Generator(device="cuda").manual_seed(R)
    x = torch.randn(4, k.num_nodes(), generator=gen, dtype=torch.float64, device="cuda")
    b = torch.randn(4, k.num_nodes(), generator=gen, dtype=torch.float64, device="cuda")
    _, dmask = k.node_info()
    b[:3, torch.tensor(dmask, device="cuda")] = 0.0
    yk, yg = k.gather(k.apply(k.scatter(x))), g.gather(g.apply(g.scatter(x)))
    rk, nk = k.residual(k.scatter(x), k.scatter(b))
    rg, ng = g.residual(g.scatter(x), g.scatter(b))
    rk, rg = k.gather(rk), g.gather(rg)
    for f in range(4):
        for a, c in ((yk, yg), (rk, rg)):
            assert float((a[f] - c[f]).abs().max()) <= TOL * float(a[f].abs().max())
    assert ng == pytest.approx(nk, rel=TOL)
    # every copy of a vertex agrees
    y = g.apply(g.scatter(x))
    assert torch.equal(g.scatter(g.gather(y)), y)
