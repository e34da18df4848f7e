"""What the solvers leave in x: a call without cycles does not write it; after a
failed HIP call it holds the cycles or iterations done."""
import os
import subprocess
import sys

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
    assert a["cycles"] == c["cycles"] and a["res_hist"] == c["res_hist"]
    # on every vertex (level 0 alone: the cycles leave anything in the padding)
    assert torch.equal(s.gather(x), t.gather(y))


# stands before the runtime in the symbol search order and returns an error from
# call number `fail` on of the host functions that the solvers call per cycle
SHIM = r"""
#include <stddef.h>
static int (*copy)(void*, const void*, size_t, int, void*);
static int (*launch)(void*, void*);
static int copies = -1, launches = -1;
void shim_set(void* c, void* l) { copy = c; launch = l; }
void shim_arm(int c, int l) { copies = c; launches = l; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) {
    return copies >= 0 && copies-- == 0 ? 1 : copy(d, s, n, k, st);
}
int hipGraphLaunch(void* g, void* s) { return launches >= 0 && launches-- == 0 ? 1 : launch(g, s); }
"""

SCRIPT = r"""
import ctypes, os, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np, torch
import workloads as W
import paper_1511_02134_amd as P
lib = {l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l}.pop()
hip = ctypes.CDLL(lib)
at = lambda f: ctypes.c_void_p(ctypes.cast(f, ctypes.c_void_p).value)
shim.shim_set(at(hip.hipMemcpyAsync), at(hip.hipGraphLaunch))
xyz, tet = W.box_mesh(1)
mesh = (xyz, tet, np.ones(len(tet)), W.face_tags(xyz, tet, 1, None))
def check(kind, done, s, call, copies, launches):
    g = torch.Generator(device="cuda").manual_seed(1)
    x0 = s.scatter(torch.randn(4, s.num_nodes(), generator=g, dtype=torch.float64, device="cuda"))
    b = s.rhs(s.scatter(torch.randn(3, s.num_nodes(), generator=g, dtype=torch.float64, device="cuda")))
    ref, x = x0.clone(), x0.clone()
    call(s, ref, b, done)
    torch.cuda.synchronize()
    shim.shim_arm(copies, launches)
    try:
        call(s, x, b, 9)
        raise SystemExit(kind + ": no error")
    except P.HHGError as e:
        assert e.status == P.HHG_EDEVICE, e
    finally:
        shim.shim_arm(-1, -1)
    torch.cuda.synchronize()
    for v in (x, ref):   # MINRES projects the pressure on its regular exit only
        s.project(v)
    d = float((s.gather(x) - s.gather(ref)).abs().max() / s.gather(ref).abs().max())
    assert d <= 1e-12, (kind, d)
    print(kind, "ok", flush=True)
solve = lambda s, x, b, k: s.solve(x, b, rtol=1e-300, max_cycles=k)
minres = lambda s, x, b, k: s.pminres(x, b, rtol=0.0, maxit=k)
# copy 0 is that of the first residual
check("copy", 2, P.Solver(*mesh, 3), solve, 2, -1)
check("copy, FP32 cycles", 2, P.Solver(*mesh, 4, precision=1, ordering=2), solve, 2, -1)
check("replay", 2, P.Solver(*mesh, 3, graphs=1), solve, -1, 2)
# an iteration's update waits for the copy of the next one
check("MINRES", 3, P.Solver(*mesh, 3, krylov=1), minres, 4, -1)
"""


def test_x_after_a_failed_call(tmp_path):
    """The failing call itself does nothing, so that the device stays as it was."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    (tmp_path / "shim.c").write_text(SHIM)
    shim = str(tmp_path / "shim.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(tmp_path / "shim.c"), "-o", shim], check=True)
    print("[gpu-case] x after a failed call", flush=True)
    r = subprocess.run([sys.executable, "-c", SCRIPT, shim, root], capture_output=True, text=True, timeout=100)
    print(r.stdout, r.stderr, flush=True)
    assert r.returncode == 0 and r.stdout.count("ok") == 4
