"""Float32 packs that hold the weights in three parts: packing, packing again and new values write the same operands, alone, together
and beside packs without the parts."""
import numpy as np
import pytest

from paper_2011_10170_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2011_10170_amd import binding
    binding.load()
    return binding


@pytest.fixture(scope="module")
def ctx(B):
    import torch
    c = B.pc_create(0, torch.cuda.current_stream().cuda_stream)
    yield c
    B.pc_destroy(c)


class _Weights:
    """Seeded weights and masks of a layer of F x C kernels."""

    def __init__(self, B, ctx, F, C, seed, dtype):
        import torch
        g = torch.Generator(device="cuda")
        g.manual_seed(seed * 1000003 + F * 1009 + C)
        self.F, self.C, self.dtype, self.lib = F, C, dtype, I.make_library(8)
        self.W = torch.randn((F, C, 9), generator=g, device="cuda")
        self.pid, self.keep = (torch.zeros((F, C), dtype=torch.uint8, device="cuda") for _ in range(2))
        B.pc_pattern_select(ctx, self.W, None, F, C, self.lib, B.PC_KEEP_PER_FILTER, I.kept_per_filter(0.4, C), B.PC_SCORE_RETAINED, self.pid, self.keep)


def _passes(B, ctx, w, pk, N, H, W, x, dy):
    import torch
    bf16 = w.dtype == B.PC_BF16
    t = torch.bfloat16 if bf16 else torch.float32
    d = B.make_desc(N, H, W, w.C, w.F, 1, w.dtype)
    y, dx = torch.full((N, H, W, w.F), float("nan"), dtype=t, device="cuda"), torch.full((N, H, W, w.C), float("nan"), dtype=t, device="cuda")
    B.pc_conv_fwd(ctx, d, pk, x.to(t), y)
    names = [B.pc_last_kernel(ctx)]
    B.pc_conv_bwd_data(ctx, d, pk, dy.to(t), dx)
    return y, dx, names + [B.pc_last_kernel(ctx)]


# blocks of 32 x 32 kernels: one, a few that are no eight, whole eights and some left, the most that have the parts; one past it
@pytest.mark.parametrize("F,C,N,H", [(32, 8, 12, 32), (31, 33, 8, 32), (130, 40, 8, 32), (65, 97, 8, 32), (199, 513, 3, 40), (320, 320, 4, 32), (1600, 64, 4, 28), (402, 256, 3, 32)])
def test_the_same_operands_whoever_writes_them(B, ctx, F, C, N, H):
    """The pack of some weights; another's, packed over with them; and one that takes the weights as new values: alone and in a call with a
    bfloat16 pack and a float32 pack without the parts. Both passes give the same bits (each is one kernel over the same operands)."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(F + C)
    x, dy = torch.randn((N, H, H, C), generator=g, device="cuda"), torch.randn((N, H, H, F), generator=g, device="cuda")
    w, other = _Weights(B, ctx, F, C, 1, B.PC_F32), _Weights(B, ctx, F, C, 2, B.PC_F32)
    half, large = _Weights(B, ctx, 40, 72, 3, B.PC_BF16), _Weights(B, ctx, 33, 3200, 4, B.PC_F32)
    sets = [w, half, large]

    def pack(v, weights=None):
        return B.pc_pack(ctx, v.W if weights is None else weights, v.pid, v.keep, v.F, v.C, v.lib, v.dtype)
    packs = {"packed": pack(w), "packed over": pack(other), "new values": pack(w, other.W), "together": pack(other), "new values together": pack(w, other.W)}
    beside = [pack(half, torch.zeros_like(half.W)), pack(large, torch.zeros_like(large.W))]
    B.pc_pack(ctx, w.W, w.pid, w.keep, F, C, w.lib, w.dtype, reuse=packs["packed over"])
    B.pc_update_values(ctx, packs["new values"], w.W)
    B.pc_pack_batch(ctx, [v.W for v in sets], [v.pid for v in sets], [v.keep for v in sets], w.lib, [packs["together"]] + beside)
    B.pc_update_values_batch(ctx, [packs["new values together"]], [w.W])
    B.pc_update_values_batch(ctx, beside + [packs["new values together"]], [half.W, large.W, w.W])
    try:
        want = _passes(B, ctx, w, packs["packed"], N, H, H, x, dy)
        parts = "true" if F * C <= 102400 else "false"
        assert any(n.startswith("pc_f32_conv_kernel<32, ") and n.endswith(", %s>" % parts) for n in want[2]), want[2]
        dense = [torch.full((F, C, 9), float("nan"), device="cuda") for _ in packs]
        for (name, pk), d in zip(packs.items(), dense):
            got = _passes(B, ctx, w, pk, N, H, H, x, dy)
            assert got[2] == want[2] and torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), name
            B.pc_unpack_dense(ctx, pk, d)
            assert torch.equal(d, dense[0]), name
        for v, pk in zip(sets[1:], beside):
            a, b = torch.empty_like(v.W), torch.empty_like(v.W)
            fresh = pack(v)
            B.pc_unpack_dense(ctx, pk, a)
            B.pc_unpack_dense(ctx, fresh, b)
            assert torch.equal(a, b)
            B.pc_packed_free(fresh)
    finally:
        for pk in list(packs.values()) + beside:
            B.pc_packed_free(pk)
