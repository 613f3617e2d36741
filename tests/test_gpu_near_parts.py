"""Near field split into parts of the near leaves' sources: trees without a
far field, so that the product is the direct sum, at sizes with one part, with
parts that begin and end inside a leaf, with more parts than leaves, and with
chunks of fewer than 64 targets.  The bars are those of the direct sum: FP64
to rounding, FP32 2e-6."""
import numpy as np
import pytest

import oracle
import synth

from gpu_common import requires_gpu, lib, dev, host, rel_l2

pytestmark = [pytest.mark.gpu, requires_gpu]
F = 0.95
BAR = {0: 1e-12, 1: 2e-6}


# panels, charges: 20 / 1 and 80 / 3 (one part), 320 / 70 (one leaf, five parts), 1,280 / 200 in 8 leaves, 5,120 in
# one leaf and in 8 (the most parts)
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("level,n_charges,ncrit",
                         [(0, 1, 99), (1, 3, 9999), (2, 70, 9999), (3, 200, 300), (4, 1500, 9999), (4, 300, 1000)])
def test_parts_sum_to_the_direct_sum(level, n_charges, ncrit, prec):
    B = lib()
    p = synth.blobby(level, n_charges=n_charges)
    g = oracle.geometry(p.verts, p.tris)
    t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=ncrit))
    assert t.info["n_far_pairs"] == 0
    rng = np.random.default_rng(5)
    x, qv = rng.normal(size=p.n_panels), rng.normal(size=p.n_charges)
    want = [oracle.apply_A(g, F, x), oracle.apply_AT(g, F, x), oracle.field_B(g, p.charge_pos, qv),
            oracle.apply_BT(g, p.charge_pos, x), oracle.apply_C(g, p.charge_pos, x), oracle.apply_CT(g, p.charge_pos, qv)]
    for op, w in enumerate(want):
        got = host(B.fmm_matvec(t, op, prec, dev(qv if op in (2, 5) else x)))
        print(f"[parts] level={level} ncrit={ncrit} prec={prec} op={op} err={rel_l2(got, w):.2e}", flush=True)
        assert rel_l2(got, w) <= BAR[prec], op
