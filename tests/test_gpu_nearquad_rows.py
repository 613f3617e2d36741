"""Near-quadrature rows of every length the kernel treats differently: none or a
few pairs, up to 16 (one load), several times 16 and not, in numbers of rows that
do not fill a wave.  The correction (product with near_quad minus product without,
trees without a far field) equals the oracle's to FP64 rounding of the product, as
in the tests of the operators."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import dev, host, lib, rel_l2, requires_gpu
from oracle import panel_integrals as PI

pytestmark = [pytest.mark.gpu, requires_gpu]

F = 1.0 - 4.0 / 80.0


# rows, pairs a row: 20 / 19; 80 / 11 to 12, 79; 320 / 3, 10 to 12, 319; 1,280 / 1 to 3, about 15
@pytest.mark.parametrize("level,nu", [(0, 16.0), (1, 2.0), (1, 16.0), (2, 1.2), (2, 2.0), (2, 16.0), (3, 1.0), (3, 2.5)])
def test_rows_of_every_length(level, nu):
    B = lib()
    p = synth.blobby(level, n_charges=2)
    g = oracle.geometry(p.verts, p.tris)
    corr = PI.kprime_correction(g, p.verts, p.tris, nu)
    t0 = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=9999))
    t1 = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=9999, near_quad=nu))
    assert t1.info["n_nearquad_pairs"] == len(corr[0]) > 0
    x = np.random.default_rng(9).normal(size=p.n_panels)
    for prec in (B.FP64, B.FP32):
        for op, tr in ((B.OP_A, False), (B.OP_AT, True)):
            d = host(B.fmm_matvec(t1, op, prec, dev(x))) - host(B.fmm_matvec(t0, op, prec, dev(x)))
            e = rel_l2(d, -F * PI.apply_correction(corr, x, g.N, transpose=tr))
            print(f"[nq-rows] level={level} nu={nu} prec={prec} op={op} pairs={len(corr[0])} err={e:.2e}", flush=True)
            assert e <= 1e-12
    B.tree_destroy(t0)
    B.tree_destroy(t1)
