"""Where hhg_solve leaves x: a call without cycles does not write it."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("R,opts", [(2, {}), (3, {"graphs": 1}), (4, {"ordering": 2, "precision": 1}),
                                    (6, {"ordering": 2, "graphs": 1})])
def test_solve_without_cycles_reports_the_residual_and_leaves_x(R, opts):
    """max_cycles = 0: r_0 of x, nothing written, copies that differ included; the
    solve after it is that of a context without the call, bit by bit."""
    import paper_1511_02134_amd as P
    print(f"[gpu-case] solve without cycles R={R} {opts}", flush=True)
    xyz, tet = W.box_mesh(1)
    mesh = (xyz, tet, np.ones(len(tet)), W.face_tags(xyz, tet, 1, None))
    s, t = P.Solver(*mesh, R, **opts), P.Solver(*mesh, R, **opts)
    g = torch.Generator(device="cuda").manual_seed(R)
    x0 = s.scatter(torch.randn(4, s.num_nodes(), generator=g, dtype=torch.float64, device="cuda"))
    b = s.rhs(s.scatter(torch.randn(3, s.num_nodes(), generator=g, dtype=torch.float64, device="cuda")))
    # every copy and the padding different
    odd = x0 + torch.rand(x0.shape, generator=g, dtype=torch.float64, device="cuda")
    x = odd.clone()
    s.solve(x, b, rtol=1e-8, max_cycles=0)
    assert torch.equal(x, odd)
    x = x0.clone()
    info = s.solve(x, b, rtol=1e-8, max_cycles=0)
    _, nrm = s.residual(x0, b)
    assert info["cycles"] == 0 and info["r0"] == pytest.approx(nrm, rel=1e-12)
    assert torch.equal(x, x0)
    y = x0.clone()
    a, c = s.solve(x, b, rtol=1e-8, max_cycles=3), t.solve(y, b, rtol=1e-8, max_cycles=3)
    assert a["cycles"] == c["cycles"] and a["res_hist"] == c["res_hist"] and torch.equal(x, y)
