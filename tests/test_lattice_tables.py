"""The lattice's tables, built from the vertices beside the corners of the cells, hold
for every vertex (host only): its record, its Dirichlet flag and the rows of B and
B^T of its class; before and after a change of viscosity."""
import numpy as np
import pytest

import paper_1511_02134_amd as P
from test_gpu_lattice_faces import _faces


@pytest.mark.parametrize("ext,R,nu_max,natural,cells", [
    ((1, 1, 1), 2, 1.0, [], False),
    ((2, 1, 3), 3, 4.0, [(1, 0)], False),
    ((3, 2, 1), 4, 1.0, [(0, 1), (1, 1), (2, 0)], True),
    ((1, 3, 2), 4, 6.0, [(0, 0), (0, 1)], True),
    ((1, 1, 1), 5, 2.0, [(2, 1)], False),
])
def test_tables_hold_for_every_vertex(ext, R, nu_max, natural, cells):
    mesh = _faces(ext, nu_max, natural, cells)
    s = P.Solver(*mesh, R, host_only=True)
    s.check_layout()
    nu = np.ascontiguousarray(mesh[2][::-1] * 3.0)
    assert P.lib.hhg_set_viscosity(s.ctx, nu.ctypes.data) == P.HHG_OK
    s.check_layout()
