"""The split of the near field into parts is a schedule, not another sum: FP32
products keep their bits for any number of parts, FP64 products agree to
rounding."""
import numpy as np
import pytest

import synth

from gpu_common import requires_gpu, lib, dev, host, rel_l2

pytestmark = [pytest.mark.gpu, requires_gpu]


def test_products_do_not_depend_on_the_parts(monkeypatch):
    B = lib()
    p = synth.blobby(5, n_charges=400)
    rng = np.random.default_rng(8)
    x, qv = rng.normal(size=p.n_panels), rng.normal(size=p.n_charges)
    outs = {}
    for parts in ("1", "2", "7", "32", "0"):                 # 0: by rule
        monkeypatch.setenv("BEMFMM_NEAR_PARTS", parts)
        t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=16, theta=0.4))
        if parts == "1":
            assert t.info["n_far_pairs"] > 0
            assert np.diff(B.tree_export(t)["near_ptr"]).max() > 64
        outs[parts] = [[host(B.fmm_matvec(t, op, prec, dev(qv if op in (2, 5) else x))) for op in range(6)]
                       for prec in (0, 1)]
        B.tree_destroy(t)
    for parts in ("2", "7", "32", "0"):
        for op in range(6):
            d = rel_l2(outs[parts][0][op], outs["1"][0][op])
            print(f"[split] parts={parts} op={op} FP64 {d:.2e}", flush=True)
            assert d <= 1e-13, (parts, op)
            assert np.array_equal(outs[parts][1][op], outs["1"][1][op]), (parts, op)
