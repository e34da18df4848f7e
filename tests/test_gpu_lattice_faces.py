"""Velocity sweeps of the lattice cycles at free vertices on the faces of the box
(natural faces), one lane per vertex and component: outflow through every face,
through several that meet in an edge, and through the faces of some cells of a
side only (free and Dirichlet vertices within a row), against cycles composed from
the entry points of the per-macro layout.  The bound is that of two orders of
summation in a cycle, 1e-11 (1e4 FP64 roundings of a row's sum)."""
import numpy as np
import pytest

import workloads as W
from test_gpu_lattice import _box, _composed

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _faces(ext, nu_max, natural, cells):
    """natural: sides as (axis, end); cells: of these sides, those of the cells
    whose index sum is even only"""
    xyz, tet, nu, tags = _box(ext, nu_max)
    for t, f in zip(*np.nonzero(tags)):
        q = xyz[np.delete(tet[t], f)]
        if cells and int(np.floor(xyz[tet[t]].mean(axis=0)).sum()) % 2:
            continue
        if any(np.all(q[:, a] == (ext[a] if e else 0)) for a, e in natural):
            tags[t, f] = W.FACE_NATURAL
    return xyz, tet, nu, tags


CASES = [
    # extents, R, largest viscosity, natural sides, some cells only, options
    ((1, 1, 1), 3, 1.0, [(0, 0)], False, {}),
    ((1, 1, 1), 4, 3.0, [(1, 1), (2, 0)], False, {"ordering": 2}),
    ((2, 1, 1), 4, 1.0, [(1, 0), (0, 1)], True, {"ordering": 2, "cycle": 1}),
    ((1, 3, 1), 4, 5.0, [(0, 1)], True, {"p_sweep": 1}),
    ((1, 2, 2), 5, 1.0, [(0, 0), (0, 1)], True, {"block_order": 0}),
    ((3, 1, 1), 5, 2.0, [(2, 1), (1, 1), (0, 0)], False, {"ordering": 2, "block_order": 2}),
    # blocks of 2 x 2 rows
    ((1, 4, 1), 7, 1.0, [(0, 1), (2, 0)], True, {"ordering": 2, "nu1": 1, "nu2": 1}),
]


@pytest.mark.parametrize("ext,R,nu_max,natural,cells,opts", CASES)
def test_cycles_with_natural_faces_equal_composed_cycles(ext, R, nu_max, natural, cells, opts):
    import paper_1511_02134_amd as P
    print(f"[gpu-case] faces {ext} R={R} natural={natural} cells={cells} {opts}", flush=True)
    s = P.Solver(*_faces(ext, nu_max, natural, cells), R, **opts)
    s.check_layout()
    gen = torch.Generator(device="cuda").manual_seed(R)
    x0 = s.scatter(torch.randn(4, s.num_nodes(), generator=gen, dtype=torch.float64, device="cuda"))
    b = s.rhs(s.scatter(torch.randn(3, s.num_nodes(), generator=gen, dtype=torch.float64, device="cuda")))
    xa, xb = x0.clone(), x0.clone()
    for _ in range(2):
        s.vcycle(xa, b)
        _composed(s, s.L, s.L, xb, b)
    ga, gb = s.gather(xa), s.gather(xb)
    assert float((ga - gb).abs().max() / gb.abs().max()) <= 1e-11
    # the free vertices of the natural sides moved, the Dirichlet ones did not
    _, dmask = s.node_info()
    d = torch.tensor(dmask, device="cuda")
    g0 = s.gather(x0)
    assert torch.equal(ga[:3, d], g0[:3, d])
    assert not torch.any(ga[:3, ~d] == g0[:3, ~d])
