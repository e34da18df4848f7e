"""Visits of a level by one workgroup use more LDS than a launch gets by default.
The limit is raised for the kernels of one and of several viscosities when the
context is made, so that a viscosity set later, which changes the kind, runs on
levels whose iterate takes more than 64 KiB (17^3 vertices in FP64)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("opts", [{}, {"precision": 1, "ordering": 2}])
def test_cycles_after_the_kind_changes(opts):
    import paper_1511_02134_amd as P
    print(f"[gpu-case] kinds {opts}", flush=True)
    xyz, tet = W.box_mesh(1)
    tags = W.face_tags(xyz, tet, 1, None)
    one, many = np.ones(len(tet)), np.linspace(0.5, 2.0, len(tet))
    R = 4
    fresh = {k: P.Solver(xyz, tet, nu, tags, R, **opts) for k, nu in (("one", one), ("many", many))}
    s = P.Solver(xyz, tet, one, tags, R, **opts)
    g = torch.Generator(device="cuda").manual_seed(1)
    x0 = s.scatter(torch.randn(4, s.num_nodes(), generator=g, dtype=torch.float64, device="cuda"))
    b = s.rhs(s.scatter(torch.randn(3, s.num_nodes(), generator=g, dtype=torch.float64, device="cuda")))
    for kind, nu in (("many", many), ("one", one), ("many", many)):
        assert P.lib.hhg_set_viscosity(s.ctx, np.ascontiguousarray(nu).ctypes.data) == P.HHG_OK
        x, y = x0.clone(), x0.clone()
        s.vcycle(x, b)
        fresh[kind].vcycle(y, b)
        assert torch.equal(s.gather(x), s.gather(y))
