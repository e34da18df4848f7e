"""The work vectors of every solver path lie inside the workspace and do not
overlap, for every combination of options that a context accepts (host only)."""
import itertools

import numpy as np
import pytest

import paper_1511_02134_amd as P
import workloads as W

COMBOS = [dict(precision=p, krylov=k, ordering=o, op=f)
          for p, k, o, f in itertools.product((0, 1), (0, 1), (0, 1, 2), (0, 1))
          if o == 0 or (k == 0 and f == 0)]


MESHES = [(1, 2, False), (1, 3, False), (2, 4, False), (1, 4, True)]
CASES = [(m, o) for m in MESHES for o in COMBOS if not (m[2] and o["ordering"] == 2)]   # red-black: Kuhn macros


@pytest.mark.parametrize("mesh,opts", CASES)
def test_work_vectors_lie_in_the_workspace(mesh, opts):
    cells, R, general = mesh
    xyz, tet = W.box_mesh(cells)
    tags = W.face_tags(xyz, tet, float(cells), None)
    phys = np.asarray(xyz, float) if general else None
    P.Solver(xyz, tet, np.ones(len(tet)), tags, R, host_only=True, phys=phys, **opts).check_layout()


@pytest.mark.parametrize("opts", [{}, {"ordering": 2}, {"precision": 1}, {"krylov": 1}, {"op": 1}, {"ordering": 1}])
def test_lattice_vectors_share_the_per_macro_ones(opts):
    """Kuhn meshes need at most one vector of the finest level (four FP64 fields) and
    9 bytes a vertex (MINRES) more than the same mesh with physical coordinates,
    which has no lattice, besides tables (a megabyte)."""
    R = 6
    xyz, tet = W.box_mesh(1)
    mesh = (xyz, tet, np.ones(len(tet)), W.face_tags(xyz, tet, 1.0, None))
    extra = {k: v for k, v in opts.items() if (k, v) != ("ordering", 2)}
    per_macro = P.plan(*mesh, R, phys=np.asarray(xyz, float), **extra)
    n = P.Solver(*mesh, R, host_only=True).vec_len()
    assert P.plan(*mesh, R, **opts) <= per_macro + (4 * 8 + 9) * n + (1 << 20)
