"""Products captured into a HIP graph after one product of the same precision:
a product after the first allocates nothing, whatever its operator.  Each graph
is replayed several times on other inputs, with the program's own products
between the replays, against the eager result."""
import gc

import numpy as np
import pytest

import synth

from gpu_common import requires_gpu, lib, dev, host

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.fixture
def no_collection():
    """A tree of an earlier test that is collected during a capture would
    synchronise the device, which ends the capture."""
    gc.collect()
    gc.disable()
    yield
    gc.enable()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("near_quad", [0.0, 2.0])
def test_capture_after_a_product_of_another_kind(prec, near_quad, no_collection):
    import torch
    B = lib()
    p = synth.blobby(4, n_charges=300)                       # 5,120 panels: the near field runs in parts
    t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(near_quad=near_quad))
    rng = np.random.default_rng(4)
    x, qv = dev(rng.normal(size=p.n_panels)), dev(rng.normal(size=p.n_charges))
    B.fmm_matvec(t, B.OP_C, prec, x)
    torch.cuda.synchronize()
    graphs = []
    for op in range(6):
        inp = qv.clone() if op in (2, 5) else x.clone()
        out = torch.empty(p.n_charges if op in (3, 4) else p.n_panels, dtype=torch.float64, device="cuda")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            B.fmm_matvec(t, op, prec, inp, y=out)
        graphs.append((op, inp, out, g))
        print(f"[capture] prec={prec} nq={near_quad} op={op} captured", flush=True)
    for rep in range(3):
        for op, inp, out, g in graphs:
            inp.copy_(dev(rng.normal(size=inp.numel())))
            g.replay()
            got = host(out)
            assert np.array_equal(got, host(B.fmm_matvec(t, op, prec, inp))), (op, rep)
    B.tree_destroy(t)


def test_capture_of_the_screened_product(no_collection):
    import torch
    B = lib()
    p = synth.blobby(4, n_charges=20)
    t = B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=32))
    rng = np.random.default_rng(4)
    z = dev(rng.normal(size=2 * p.n_panels))
    out = torch.empty_like(z)
    B.lpb_matvec(t, 0.2, z)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.lpb_matvec(t, 0.2, z, y=out)
    for rep in range(3):
        z.copy_(dev(rng.normal(size=z.numel())))
        g.replay()
        got = host(out)
        assert np.array_equal(got, host(B.lpb_matvec(t, 0.2, z))), rep
    B.tree_destroy(t)
