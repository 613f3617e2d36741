"""GMRES cycles whose steps change from the fused kernels of short vectors and
few basis vectors to the separate ones, restarts, and combinations of more basis
vectors than travel as kernel arguments (64), against the dense oracle's solve.
The tolerance is below what the Givens estimate reaches in the steps given (it
falls by a factor of about 20 a step on these surfaces, past rounding), so that
the steps are taken.  The trees have no far field; A's smallest singular value is
about 1 - f = 0.05, so a residual of 1e-10 leaves x within 1e-8."""
import pytest

import oracle
import synth

from gpu_common import requires_gpu, lib, dev, host, rel_l2

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("level,restart,maxit", [(0, 33, 33), (2, 32, 66), (2, 64, 64), (2, 70, 70), (3, 100, 100),
                                                 (2, 70, 150)])
def test_long_cycles_match_oracle(level, restart, maxit):
    B = lib()
    p = synth.blobby(level, n_charges=12)
    g = oracle.geometry(p.verts, p.tris)
    t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=9999))
    x, info = B.solve_bem(t, dev(p.q), tol=1e-200, maxit=maxit, restart=restart, precision=B.FP64, raise_on_noconv=False)
    want, _ = oracle.solve(g, p.charge_pos, p.q, 4.0, 80.0, tol=1e-12)
    e = rel_l2(host(x), want)
    print(f"[krylov] level={level} restart={restart} iters={info.iters} err={e:.2e}", flush=True)
    if level > 0:                                          # 20 panels: the Krylov space can end before
        assert info.iters == maxit
    assert e <= 1e-8


@pytest.mark.parametrize("level,restart", [(1, 1), (2, 3)])
def test_restarted_cycles_match_oracle(level, restart):
    B = lib()
    p = synth.blobby(level, n_charges=12)
    g = oracle.geometry(p.verts, p.tris)
    t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=9999))
    x, info = B.solve_bem(t, dev(p.q), tol=1e-10, maxit=2000, restart=restart, precision=B.FP64)
    want, _ = oracle.solve(g, p.charge_pos, p.q, 4.0, 80.0, tol=1e-12)
    assert info.iters > restart
    assert rel_l2(host(x), want) <= 1e-8
