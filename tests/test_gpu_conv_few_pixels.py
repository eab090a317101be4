"""The forward / backward-data kernel for few pixels and many channels (override codes 51 to 54; up to 512 reduction channels): element by element against the oracle, at maps of one row or column, tiles across images, a last tile of few pixels, reduction
channels that fill no chunk or wavefront, and every turn of a pixel's pieces; and the fused steps."""
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


SHAPES = [
    (1, 1, 1, 32, 32, 1),         # one pixel
    (3, 1, 5, 64, 96, 1),         # maps of one row and of one column; pieces turned by 8 and by 4
    (5, 7, 1, 96, 64, 1),
    (9, 2, 2, 128, 160, 1),       # many images in a tile
    (1, 14, 14, 512, 256, 1),     # the largest reduction
    (2, 7, 9, 288, 512, 1),       # a second chunk for one wavefront only
    (2, 9, 8, 8, 24, 1),          # one group of channels: most of a chunk is zeros
    (3, 6, 5, 264, 136, 1),       # the last chunk has 8 channels, in the second round of wavefronts
    (1, 11, 13, 232, 488, 1),
    (1, 28, 27, 256, 288, 1),
    (4, 5, 6, 320, 416, 1)]


@pytest.mark.parametrize("cfg", [51, 52, 53, 54])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_element(B, ctx, oracle, cfg, shape):
    B.pc_set_plan_override(ctx, cfg, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_MFMA, ("few", cfg))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("cfg", [51, 52, 53, 54])
@pytest.mark.parametrize("dims", [(1, 14, 14, 512, 512), (3, 9, 7, 256, 96)])
def test_fused_steps(B, ctx, cfg, dims):
    import torch
    from tests._harness import Case, GpuLayer
    layer = I.Layer(*dims, 1)
    g = GpuLayer(B, ctx, Case(layer, "bf16", 8, I.kept_per_filter(0.3, layer.C), tag=("few", "fused")))
    try:
        B.pc_set_plan_override(ctx, cfg, 0)
        y, yr = (torch.full((layer.N, layer.Ho, layer.Wo, layer.F), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        dx, dr = (torch.full((layer.N, layer.H, layer.W, layer.C), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, y)
        B.pc_conv_fwd_relu(ctx, g.desc, g.pk, g.x, yr)
        B.pc_conv_bwd_data(ctx, g.desc, g.pk, g.dy, dx)
        B.pc_conv_bwd_data_relu(ctx, g.desc, g.pk, g.dy, g.x, dr)
        assert "pc_mfma_conv_deep_kernel" in B.pc_last_kernel(ctx)
        assert torch.equal(yr, torch.where(y > 0, y, torch.zeros_like(y)))
        assert torch.equal(dr, torch.where(g.x > 0, dx, torch.zeros_like(dx)))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        g.close()
