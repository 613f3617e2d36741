"""Products on a card with little free memory.  The memory is held by torch
tensors, sized from what the same product on the same tree took before; nothing
but the library's own allocations meets the limit, and it reports them."""
import numpy as np
import pytest

import synth

from gpu_common import requires_gpu, lib, dev, host

pytestmark = [pytest.mark.gpu, requires_gpu]
MB = 1 << 20


class Low:
    """Holds all but `left` bytes of the card's free memory."""

    def __init__(self, left):
        self.left = left

    def __enter__(self):
        import torch
        lib().release_cache()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        self.blocks = []
        for _ in range(8):                                 # the free amount settles after the first
            over = torch.cuda.mem_get_info()[0] - int(self.left)
            if over < 4 * MB:
                break
            self.blocks.append(torch.empty(over, dtype=torch.uint8, device="cuda"))
        # both allocators round up; the cases have 100 MB and more to spare on either side
        assert abs(torch.cuda.mem_get_info()[0] - self.left) < 64 * MB
        print(f"[memory] {torch.cuda.mem_get_info()[0] / MB:.0f} MB left", flush=True)

    def __exit__(self, *exc):
        import torch
        self.blocks.clear()
        torch.cuda.empty_cache()


def _build(B):
    p = synth.blobby(5, n_charges=200)                     # 20,480 panels
    return p, B.build_tree(p.verts, p.tris, p.charge_pos, B.Params(ncrit=16, theta=0.3))


def _first_product(B, t, prec, x):
    """Its result and the device memory it took."""
    import torch
    B.release_cache()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    y = host(B.fmm_matvec(t, B.OP_A, prec, x))
    return y, free - torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("prec", [0, 1])
def test_product_after_one_that_found_no_memory(prec):
    """ENOMEM leaves the tree valid: with the memory back, the next product is
    that of a tree that never met the limit."""
    B = lib()
    p, t = _build(B)
    x = dev(np.random.default_rng(2).normal(size=p.n_panels))
    want, used = _first_product(B, t, prec, x)
    B.tree_destroy(t)
    assert used >= 300 * MB
    p, t = _build(B)
    y = torch_empty(p.n_panels)
    with Low(used / 4):
        with pytest.raises(B.BemfmmError) as ei:
            B.fmm_matvec(t, B.OP_A, prec, x, y=y)
        assert ei.value.code == 2
    np.testing.assert_array_equal(host(B.fmm_matvec(t, B.OP_A, prec, x)), want)
    B.tree_destroy(t)


def test_near_field_without_room_for_its_parts(monkeypatch):
    """FP32 leaf totals are scratch that only a near field in parts needs: with
    room for half of them the product runs whole chunks, to the same bits."""
    B = lib()
    monkeypatch.setenv("BEMFMM_NEAR_PARTS", "4")
    p, t = _build(B)
    x = dev(np.random.default_rng(2).normal(size=p.n_panels))
    near = np.diff(B.tree_export(t)["near_ptr"]).max()
    leaf = t.info["n_leaves"] * int(near) * 3 * 64 * 4
    assert 100 * MB <= leaf <= 1024 * MB
    want, used = _first_product(B, t, B.FP32, x)
    B.tree_destroy(t)
    p, t = _build(B)
    y = torch_empty(p.n_panels)
    with Low(used - leaf / 2):
        got = [host(B.fmm_matvec(t, op, B.FP32, x, y=y)) for op in (B.OP_A, B.OP_AT, B.OP_A)]
    np.testing.assert_array_equal(got[0], want)
    np.testing.assert_array_equal(got[2], want)
    np.testing.assert_array_equal(host(B.fmm_matvec(t, B.OP_AT, B.FP32, x)), got[1])
    B.tree_destroy(t)


def torch_empty(n):
    import torch
    return torch.empty(n, dtype=torch.float64, device="cuda")
