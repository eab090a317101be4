"""GPU parity of the first-layer kernels (stride 1, at most 4 input channels): every output element of the three
passes against the oracle, on shapes with ragged rows, columns and tiles, 1 to 4 input channels and 1 to 4 row tiles
of 32 filters; the fused ReLU of the forward launch; and that the automatic choice really takes these kernels."""
import numpy as np
import pytest

from paper_2011_10170_amd import inputs as I
from tests.test_gpu_parity import run_case

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

# (N, H, W, C, F, stride): the backward-data kernel takes 32 and 64 filters, the forward kernel up to 128
FIRST_LAYER_SHAPES = [
    (2, 9, 37, 3, 64, 1),       # ragged rows and columns
    (3, 16, 32, 1, 32, 1),      # one channel, one row tile
    (1, 8, 40, 4, 96, 1),       # four channels, three row tiles (backward-data on the general kernels)
    (2, 17, 33, 2, 64, 1),
    (1, 5, 300, 3, 128, 1),     # two column tiles, four row tiles
    (4, 32, 32, 3, 64, 1),      # the CIFAR first layer
    (1, 1, 1, 3, 32, 1),        # a single pixel
]


@pytest.mark.parametrize("keep", [0.3, 1.0])
@pytest.mark.parametrize("shape", FIRST_LAYER_SHAPES)
def test_first_layer_passes(B, ctx, oracle, shape, keep):
    run_case(B, ctx, oracle, shape, "bf16", 8, keep, B.PC_VARIANT_MFMA, ("first_layer", keep))


@pytest.mark.parametrize("shape", [(2, 9, 37, 3, 64, 1), (3, 16, 32, 1, 32, 1)])
def test_first_layer_kernels_forced(B, ctx, oracle, shape):
    """Override code 23 fails rather than falling back to another kernel."""
    B.pc_set_plan_override(ctx, 23, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.4, B.PC_VARIANT_MFMA, "first_layer_forced")
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


def test_first_layer_kernels_are_the_automatic_choice_and_fuse_the_relu(B, ctx):
    import torch
    from tests._harness import Case, GpuLayer
    layer = I.Layer(3, 20, 45, 3, 64, 1)
    case = Case(layer, "bf16", 8, I.kept_per_filter(0.4, layer.C), tag="first_layer_auto")
    g = GpuLayer(B, ctx, case)
    try:
        L = layer
        y = torch.empty((L.N, L.Ho, L.Wo, L.F), dtype=torch.bfloat16, device="cuda")
        a = torch.full_like(y, float("nan"))
        dx = torch.empty((L.N, L.H, L.W, L.C), dtype=torch.bfloat16, device="cuda")
        dz = torch.full_like(dx, float("nan"))
        B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, y)
        assert B.pc_last_kernel(ctx).startswith("pc_thin_fwd_kernel")
        B.pc_conv_fwd_relu(ctx, g.desc, g.pk, g.x, a)
        B.pc_conv_bwd_data(ctx, g.desc, g.pk, g.dy, dx)
        assert B.pc_last_kernel(ctx).startswith("pc_thin_bwd_data_kernel")
        B.pc_conv_bwd_data_relu(ctx, g.desc, g.pk, g.dy, g.x, dz)
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.int16), torch.where(y > 0, y, torch.zeros_like(y)).view(torch.int16))
        assert torch.equal(dz.view(torch.int16), torch.where(g.x > 0, dx, torch.zeros_like(dx)).view(torch.int16))
        # a forced general kernel gives the same values up to the float32 order of additions
        from tests._harness import rel_l2, from_dev_f32
        B.pc_set_plan_override(ctx, 6, 0)
        yg = torch.empty_like(y)
        dxg = torch.empty_like(dx)
        B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, yg)
        assert B.pc_last_kernel(ctx).startswith("pc_mfma_conv_kernel")
        B.pc_conv_bwd_data(ctx, g.desc, g.pk, g.dy, dxg)
        torch.cuda.synchronize()
        assert rel_l2(from_dev_f32(y), from_dev_f32(yg)) <= 3e-3 and rel_l2(from_dev_f32(dx), from_dev_f32(dxg)) <= 3e-3
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        g.close()


@pytest.mark.parametrize("shape", [
    (1, 1, 2, 4, 8, 1), (40, 2, 2, 3, 16, 1), (2, 64, 31, 2, 48, 1), (1, 224, 9, 3, 136, 1), (3, 9, 11, 3, 24, 2), (7, 5, 3, 4, 64, 2), (5, 33, 35, 1, 72, 2),
    (9, 32, 32, 3, 32, 1)])
def test_backward_weight_of_few_channels(B, ctx, oracle, shape):
    """Rows across images, columns past the map, blocks of 16 and of 64 filters that are not full, both strides, and x at an address that is a multiple
    of 2 only (its last pixel is read with the bytes before it)."""
    import torch
    from tests._harness import Case, GpuLayer
    run_case(B, ctx, oracle, shape, "bf16", 8, 0.5, B.PC_VARIANT_MFMA, "few_channels")
    assert B.pc_last_kernel(ctx).startswith("pc_thin_wgrad_kernel")
    g = GpuLayer(B, ctx, Case(I.Layer(*shape), "bf16", 8, I.kept_per_filter(0.5, shape[3]), tag=("few", shape)))
    try:
        want = g.bwd_weight()[0]
        moved = torch.zeros(g.x.numel() + 8, dtype=g.x.dtype, device="cuda")
        for off in (1, 2, 3):
            moved.fill_(float("nan"))
            moved[off:off + g.x.numel()].copy_(g.x.reshape(-1))
            got = torch.full((g.nnzk, 4), float("nan"), device="cuda")
            B.pc_conv_bwd_weight(ctx, g.desc, g.pk, moved[off:], g.dy, got)
            assert B.pc_last_kernel(ctx).startswith("pc_thin_wgrad_kernel")
            assert np.array_equal(got.cpu().numpy(), want)
    finally:
        g.close()


@pytest.mark.parametrize("shape", [(2, 9, 37, 3, 8, 1), (1, 5, 300, 4, 24, 1), (3, 16, 32, 1, 56, 1), (2, 17, 33, 2, 104, 1)])
def test_forward_with_a_row_tile_that_is_not_full(B, ctx, oracle, shape):
    """Filter counts that are multiples of 8 only: nothing is stored past the last filter, with and without the fused ReLU."""
    import torch
    from tests._harness import Case, GpuLayer, Guarded
    run_case(B, ctx, oracle, shape, "bf16", 8, 0.4, B.PC_VARIANT_MFMA, "first_layer_rows")
    L = I.Layer(*shape)
    g = GpuLayer(B, ctx, Case(L, "bf16", 8, I.kept_per_filter(0.4, L.C), tag=("rows", shape)))
    try:
        y, a = (Guarded(L.N * L.Ho * L.Wo * L.F, torch.bfloat16) for _ in range(2))
        B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, y.ptr)
        assert B.pc_last_kernel(ctx).startswith("pc_thin_fwd_kernel")
        B.pc_conv_fwd_relu(ctx, g.desc, g.pk, g.x, a.ptr)
        assert B.pc_last_kernel(ctx).startswith("pc_thin_fwd_kernel")
        torch.cuda.synchronize()
        assert y.margins_intact() and a.margins_intact()
        assert torch.equal(a.body.view(torch.int16), torch.where(y.body > 0, y.body, torch.zeros_like(y.body)).view(torch.int16))
    finally:
        g.close()


@pytest.mark.parametrize("shape", [(3, 9, 11, 3, 40, 1), (1, 224, 9, 3, 136, 1), (2, 64, 31, 2, 48, 1), (5, 33, 35, 1, 72, 2), (7, 5, 3, 4, 64, 2), (9, 32, 32, 3, 32, 1)])
def test_backward_weight_of_few_channels_in_a_group(B, ctx, oracle, shape):
    """Behind the workgroups of other layers in their launch (more than 32 filters) and in its own: the sums of a call of its own, of which
    every workgroup takes the same tiles."""
    import torch
    from tests._harness import Case, GpuLayer, rel_l2
    shapes = [(2, 14, 14, 64, 64, 1), shape, (3, 8, 8, 64, 128, 1)]
    gs = [GpuLayer(B, ctx, Case(I.Layer(*s), "bf16", 8, I.kept_per_filter(0.5, s[3]), tag=("group", s))) for s in shapes]
    try:
        want = gs[1].bwd_weight()[0]
        assert B.pc_last_kernel(ctx).startswith("pc_thin_wgrad_kernel")
        for _ in range(2):
            outs = [torch.full((g.nnzk, 4), float("nan"), device="cuda") for g in gs]
            B.pc_conv_bwd_weight_batch(ctx, [g.desc for g in gs], [g.pk for g in gs], [g.x for g in gs], [g.dy for g in gs], outs)
            assert B.pc_last_kernel(ctx).startswith("pc_mfma_wgrad_dma_group_kernel")
            torch.cuda.synchronize()
            assert np.array_equal(outs[1].cpu().numpy(), want)
            for g, o in zip(gs, outs):
                assert rel_l2(o.cpu().numpy(), g.bwd_weight()[0]) <= 1e-5
    finally:
        for g in gs:
            g.close()
