"""Per-level M2M and L2L products at the orders and level sizes where their
kernel changes: 1 to 3 column tiles (orders 3 and 6), 4 (order 8: levels up to 40
tiles of 64 rows, and longer), 6 to 8 (orders 9 to 11: up to 200 tiles, and longer).
The tree has levels of a few to some 20,000 cells.  Multipoles of sampled cells
equal their definition to rounding (M2M is exact); the product, which the L2L
enters, meets the truncation error of its order against the dense oracle."""
import numpy as np
import pytest

import oracle
import oracle.harmonics as H
import oracle.tree as OT
import synth

from gpu_common import requires_gpu, lib, dev, host, rel_l2

pytestmark = [pytest.mark.gpu, requires_gpu]
BAR = {3: 3e-2, 6: 1e-3, 8: 1e-4, 9: 1e-4, 10: 1e-5, 11: 1e-5}


@pytest.fixture(scope="module")
def case():
    p = synth.blobby(5, n_charges=20)                       # 20,480 panels
    g = oracle.geometry(p.verts, p.tris)
    x = np.random.default_rng(3).normal(size=p.n_panels)
    return p, g, x, oracle.apply_A(g, 0.95, x)


@pytest.mark.parametrize("prec,tol", [(0, 1e-11), (1, 2e-6)])
@pytest.mark.parametrize("order", sorted(BAR))
def test_level_products(case, order, prec, tol):
    p, g, x, want = case
    B = lib()
    t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=1, p=order))
    y = host(B.fmm_matvec(t, B.OP_A, prec, dev(x)))
    Mg, ex = B.debug_expansions(t, prec, 0), B.tree_export(t)
    lo, side, lev = np.array(t.info["lo"]), t.info["side"], ex["cell_level"]
    cells = [int((lev == l).sum()) for l in range(t.info["leaf_level"] + 1)]
    print(f"[level] order={order} prec={prec} cells={cells} err={rel_l2(y, want):.2e}", flush=True)
    assert max(cells) > 200 * 64 + 8 * 64 and any(40 * 64 + 8 * 64 < c < 200 * 64 for c in cells)
    w = g.a * x
    for l in range(2, t.info["leaf_level"]):
        sel = np.nonzero(lev == l)[0]
        for c in sel[:: max(1, len(sel) // 12)]:
            b, e = ex["cell_range"][c][:2]
            if e == b:
                continue
            s = side / (1 << l)
            X = lo + (OT.deinterleave(np.array([ex["cell_key"][c]], dtype=np.int64), l)[0] + 0.5) * s
            idx = ex["panel_perm"][b:e]
            m = H.p2m(g.c[idx], w[idx], X, s, order)
            assert np.abs(Mg[c] - m).max() <= tol * np.abs(m).max(), (l, c)
    assert rel_l2(y, want) <= BAR[order]
    B.tree_destroy(t)
