"""Arnoldi steps of short vectors (one workgroup and several, rows that do not
fill one), restarts that add to the solution, and more basis vectors than the
combination takes as arguments, against the dense oracle's solve.  The trees
have no far field, so the operators agree to rounding; A's smallest singular
value is about 1 - f = 0.05, so a residual of 1e-10 leaves x within 1e-8."""
import pytest

import oracle
import synth

from gpu_common import requires_gpu, lib, dev, host, rel_l2

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("level,restart,maxit,tol",
                         [(0, 30, 200, 1e-10), (1, 1, 2000, 1e-10), (2, 3, 500, 1e-10), (3, 30, 200, 1e-10),
                          (2, 70, 70, 1e-30)])
def test_short_vector_solve_matches_oracle(level, restart, maxit, tol):
    B = lib()
    p = synth.blobby(level, n_charges=12)
    g = oracle.geometry(p.verts, p.tris)
    t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=9999))
    x, info = B.solve_bem(t, dev(p.q), tol=tol, maxit=maxit, restart=restart, precision=B.FP64, raise_on_noconv=False)
    want, _ = oracle.solve(g, p.charge_pos, p.q, 4.0, 80.0, tol=1e-12)
    e = rel_l2(host(x), want)
    print(f"[arnoldi] level={level} restart={restart} iters={info.iters} err={e:.2e}", flush=True)
    assert e <= 1e-8
