"""t_solve_ms leaves out no more of a call than the first residual and a
synchronisation: the conversions of x and b to the layout of the cycles are in it
(1.4 ms for 17 M vertices on the way in)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _ms(call):
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    a.record()
    r = call()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b), r


def test_solve_time_holds_the_conversions():
    import paper_1511_02134_amd as P
    print("[gpu-case] solve time R=8", flush=True)
    xyz, tet = W.box_mesh(1)
    s = P.Solver(xyz, tet, np.ones(len(tet)), W.face_tags(xyz, tet, 1, None), 8, ordering=2)
    x, b = s.vector(), s.rhs(torch.ones(3, s.vec_len(), dtype=torch.float64, device="cuda"))
    r, nrm = s.vector(), torch.zeros(1, dtype=torch.float64, device="cuda")
    rest, first = [], []
    for _ in range(6):
        x.zero_()
        t, info = _ms(lambda: s.solve(x, b, rtol=1e-300, max_cycles=1))
        rest.append(t - info["t_solve_ms"])
        first.append(_ms(lambda: s.residual_noalloc(x, b, r, nrm))[0])
    print(f"outside t_solve_ms {min(rest):.3f} ms, a residual {min(first):.3f} ms", flush=True)
    assert min(rest) <= min(first) + 0.3
