"""The forward / backward-data kernel that keeps a layer's weights in LDS (override code 50; up to 64 channels on both sides): element by
element against the oracle at the edges of its tiles, and layers of many tiles per workgroup, with the fused ReLU steps, against a kernel
of another family."""
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


@pytest.mark.parametrize("shape", [
    (1, 1, 1, 8, 8, 1),          # one pixel, one group of channels
    (3, 2, 3, 8, 16, 1),         # rows of several images in a tile
    (1, 33, 47, 40, 64, 1),      # a last chunk of 8 channels, a row and columns past the last tile
    (2, 31, 17, 56, 24, 1),      # 24 channels in the last chunk; one row short of a tile; 32 channels and 64 in turn
    (7, 16, 9, 48, 32, 1),       # images that divide a tile
    (5, 13, 8, 64, 56, 1),       # images that do not
    (20, 64, 65, 32, 64, 1),     # more tiles than workgroups
    (9, 96, 95, 64, 40, 1)])
def test_every_element(B, ctx, oracle, shape):
    from tests._harness import Case, GpuLayer
    layer = I.Layer(*shape)
    B.pc_set_plan_override(ctx, 50, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_MFMA, "resident")
        g = GpuLayer(B, ctx, Case(layer, "bf16", 8, I.kept_per_filter(0.3, layer.C), tag="resident"), variant=B.PC_VARIANT_MFMA)
        for run, channels in ((g.fwd, layer.F), (g.bwd_data, layer.C)):      # (two fragments of 16 output channels a wavefront, or four)
            run()
            assert B.pc_last_kernel(ctx).startswith("pc_mfma_conv_keep_kernel<%d, " % (2 if channels <= 32 else 4)), B.pc_last_kernel(ctx)
        g.close()
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("dims", [(16, 56, 56, 64, 64), (33, 100, 99, 64, 24), (70, 61, 60, 24, 64), (90, 50, 51, 32, 32), (64, 35, 29, 8, 40)])
def test_many_tiles_per_workgroup(B, ctx, dims):
    """The buffers run on from tile to tile at every offset, while finished tiles leave. Two kernels round sums that they add in another
    order: one unit in the last place of bfloat16, 2^-7 of the value at most, or the addition's error where terms cancel."""
    import torch
    from tests._harness import Case, GpuLayer
    layer = I.Layer(*dims, 1)
    g = GpuLayer(B, ctx, Case(layer, "bf16", 8, I.kept_per_filter(0.3, layer.C), tag=("resident", "tiles")))
    try:
        out = []
        for code in (50, 20):
            B.pc_set_plan_override(ctx, code, 0)
            y, yr = (torch.full((layer.N, layer.Ho, layer.Wo, layer.F), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
            dx, dr = (torch.full((layer.N, layer.H, layer.W, layer.C), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
            B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, y)
            B.pc_conv_fwd_relu(ctx, g.desc, g.pk, g.x, yr)
            B.pc_conv_bwd_data(ctx, g.desc, g.pk, g.dy, dx)
            B.pc_conv_bwd_data_relu(ctx, g.desc, g.pk, g.dy, g.x, dr)
            assert ("pc_mfma_conv_keep_kernel" in B.pc_last_kernel(ctx)) == (code == 50)
            assert torch.equal(yr, torch.where(y > 0, y, torch.zeros_like(y)))
            assert torch.equal(dr, torch.where(g.x > 0, dx, torch.zeros_like(dx)))
            out.append((y.double(), dx.double()))
        for a, b in zip(*out):
            assert bool((a - b).abs().le(2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 2.0 ** -12 * b.abs().max()).all())
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        g.close()
