"""MINRES on contexts whose cycles run in FP32 (precision = 1): its vectors and
velocity cycles are FP64 whatever the precision of the cycles, so the iterates
are those of the oracle to the bounds of the FP64 contexts' tests (1e-11 of the
history, 1e-9 of the iterate after a few iterations), before and after a solve
in mixed precision on the same context."""
import numpy as np
import pytest

import workloads as W
from oracle import UMG, build_hierarchy
from oracle.krylov import StokesKrylov

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("cid,R,iters", [(1, 2, 3), (1, 3, 3), (4, 4, 5), (5, 4, 4)])
def test_pminres_of_a_mixed_context_matches_oracle(cid, R, iters):
    import paper_1511_02134_amd as P
    print(f"[gpu-case] PMINRES, mixed context, config {cid} R={R}", flush=True)
    cfg = W.WORKLOADS[cid].with_R(R)
    xyz, tet, nu, tags = cfg.mesh()
    s = P.Solver(xyz, tet, nu, tags, R, krylov=1, precision=1)
    s.check_layout()   # every vector inside the workspace, before anything runs
    H = build_hierarchy(xyz, tet, nu, tags, R)
    lv = H.finest
    b = UMG(H).rhs(cfg.forcing_field() + W.nodal_noise(lv.N, 5, 1.0))
    x0 = np.random.default_rng(6).normal(size=(4, lv.N))
    x0[:3, lv.dirichlet] = cfg.dirichlet_field()[:, lv.dirichlet]
    xo, ho = StokesKrylov(H, 1, 1).pminres(x0, b, rtol=0.0, maxit=iters)
    xd0, bd = s.scatter(torch.tensor(x0, device="cuda")), s.scatter(torch.tensor(b, device="cuda"))
    for again in range(2):
        xd = xd0.clone()
        info = s.pminres(xd, bd, rtol=0.0, maxit=iters)
        xg = s.gather(xd).cpu().numpy()
        assert info["cycles"] == iters
        assert np.abs(np.array(info["res_hist"]) - np.array(ho)).max() / ho[0] < 1e-11
        assert np.abs(xg - xo).max() / np.abs(xo).max() < 1e-9
        if not again:
            s.solve(xd, bd, rtol=1e-8, max_cycles=3)
