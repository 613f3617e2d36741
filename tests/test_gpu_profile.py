"""Stage times of products with near quadrature: the p2p stage holds the whole
near field, the corrections of the close pairs with the direct sums."""
import pytest

import synth

from gpu_common import requires_gpu, lib, dev, host

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("prec", [0, 1])
def test_p2p_stage_holds_the_near_quadrature(prec, monkeypatch):
    """nu = 16 corrects some 500 pairs a panel, 12 bytes each, as much time as
    the 4,000 direct pairs take; in line, the two stages do not share the chip."""
    import numpy as np
    B = lib()
    monkeypatch.setenv("BEMFMM_CONCURRENT_P2P", "0")
    p = synth.blobby(5, n_charges=20)                       # 20,480 panels
    x = dev(np.random.default_rng(1).normal(size=p.n_panels))
    ms = {}
    for nu in (0.0, 16.0):
        t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(near_quad=nu))
        host(B.fmm_matvec(t, B.OP_A, prec, x))
        B.profile(t, True)
        for _ in range(20):
            B.fmm_matvec(t, B.OP_A, prec, x)
        total, count = B.profile_get(t, f"p2p/{B.OP_A}/{prec}")
        assert count == 20
        ms[nu] = total / count
        print(f"[profile] prec={prec} nu={nu} pairs={t.info['n_nearquad_pairs']} p2p {1e3 * ms[nu]:.1f} us", flush=True)
        B.tree_destroy(t)
    assert ms[16.0] >= 1.15 * ms[0.0]
