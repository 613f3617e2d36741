"""The split of the near field into parts is a schedule, not another sum.

FP32 products keep their bits for any number of parts.  In FP64 the parts'
compensated sums, with the rests that one number does not hold, add up to what
one compensated sum over the whole near list gives: where hundreds of terms
cancel, the two agree to roundings of single terms."""
import numpy as np
import pytest

import synth
from oracle.tree import interleave, quantise

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


# 20,480 panels: chunks of one lane group; 1,280 panels: about 20 lane groups a chunk
@pytest.mark.parametrize("level,ncrit", [(5, 64), (3, 5)])
def test_fp64_parts_keep_the_compensation(level, ncrit, monkeypatch):
    """Two charges in the middle of every cell of an 8^3 lattice around the
    surface, of opposite sign in the two halves of the near list and values for
    which the field at one panel cancels, as potential (C^T) and as normal
    gradient (B).  Every term is at most 2.5 in size; a compensated sum rounds
    each once more, so two of them over n terms differ by about sqrt(2 n) u, 30 u
    for the 400 terms here, u = 2^-53, and the bar is 64 u times the largest
    term.  Parts that add plain sums are off by hundreds of u."""
    B = lib()
    p = synth.blobby(level, n_charges=1)
    t0 = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=ncrit, theta=0.3))
    assert t0.info["leaf_level"] == 3
    lo, side = np.asarray(t0.info["lo"]), t0.info["side"]
    B.tree_destroy(t0)
    s = side / 8
    k = np.arange(8)
    cell = np.stack(np.meshgrid(k, k, k, indexing="ij"), -1).reshape(-1, 3)
    rng = np.random.default_rng(3)
    pos = (lo + (np.repeat(cell, 2, 0) + rng.uniform(0.3, 0.7, size=(2 * len(cell), 3))) * s)
    c = p.verts[p.tris].mean(1)
    pos = pos[np.argsort(interleave(quantise(pos, lo, side)))]  # the order of the near lists
    targets = rng.choice(p.n_panels, 6, replace=False)
    worst = {}
    trees = {}
    for parts in ("1", "32"):
        monkeypatch.setenv("BEMFMM_NEAR_PARTS", parts)
        trees[parts] = B.build_tree(p.verts, p.tris, pos, B.Params(ncrit=ncrit, theta=0.3))
        assert trees[parts].info["leaf_level"] == 3
        assert abs(trees[parts].info["side"] - side) <= 1e-9 * side
        B.debug_record(trees[parts], True)
        B.fmm_matvec(trees[parts], B.OP_CT, B.FP64, dev(np.zeros(len(pos))))  # the switch is read here
    for op, name in ((B.OP_CT, "CT"), (B.OP_B, "B")):
        for t in targets:
            d = c[t] - pos
            r = np.linalg.norm(d, axis=1)
            tc = np.floor((c[t] - lo) / s)
            near = (np.abs(np.floor((pos - lo) / s) - tc) ** 2).sum(1) <= 33
            q = np.zeros(len(pos))
            idx = np.nonzero(near)[0]
            if name == "CT":
                term = (1.0 / r)[idx]
                rows = term[None]
            else:
                term = (np.abs(d).max(1) / r ** 3)[idx]
                rows = (d / r[:, None] ** 3)[idx].T
            sign = np.where(np.arange(len(idx)) < len(idx) // 2, 1.0, -1.0)
            w = sign * rng.uniform(1, 2, len(idx)) / term
            G = rows * (1.0 / term)                             # in units of the terms
            z = w * term
            z -= G.T @ np.linalg.solve(G @ G.T, G @ z)          # every component cancels
            q[idx] = z / term
            f = {}
            for parts, tree in trees.items():
                B.fmm_matvec(tree, op, B.FP64, dev(q))
                f[parts] = B.debug_fields(tree, B.FP64, p.n_panels)[0][t] * 4 * np.pi
            e = abs(f["32"] - f["1"]) / np.abs(z).max() * 2.0 ** 53
            print(f"[split] {name} level={level} near={len(idx)} diff {e:.1f} u, sum {f['1']:.2e}", flush=True)
            worst[name] = max(worst.get(name, 0.0), e)
    for t in trees.values():
        B.tree_destroy(t)
    for name, e in worst.items():
        assert e <= 64, (name, e)
