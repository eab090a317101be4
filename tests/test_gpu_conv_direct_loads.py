"""The forward / backward-data kernels that load both operands straight to LDS (override codes 40 to 49; 37 and 38 for stride-2
backward-data), element by element against the oracle, at the edges of their tiles: rows that run across images, columns past the map, a last chunk of 8, 16 or 24 channels, partial row tiles, and lists of tiles that
continue in narrower ones."""
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
    (1, 1, 1, 8, 8, 1),          # one pixel, one group of channels
    (3, 2, 3, 8, 16, 1),         # rows of several images in a tile
    (1, 33, 47, 40, 72, 1),      # a last chunk of 8 channels, a row and columns past the last tile
    (2, 31, 17, 56, 24, 1),      # 24 channels in the last chunk; one row short of a tile
    (7, 16, 9, 80, 136, 1),      # images that divide a tile, 16 channels in the last chunk
    (5, 13, 8, 64, 200, 1),      # images that do not
    (1, 64, 5, 32, 64, 1),       # whole chunks and row tiles
    (9, 96, 95, 16, 200, 1),     # more tiles than workgroups: the list ends in narrower tiles
    (6, 96, 95, 40, 264, 1),
]


@pytest.mark.parametrize("cfg", [40, 41, 42, 43, 45, 46])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_element(B, ctx, oracle, cfg, shape):
    B.pc_set_plan_override(ctx, cfg, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_MFMA, ("direct", cfg))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("cfg", [47, 48, 49, 37, 38])
@pytest.mark.parametrize("shape", [s[:5] + (2,) for s in SHAPES] + [(70, 4, 4, 72, 64, 2), (5, 32, 32, 64, 64, 2), (3, 64, 66, 136, 40, 2)])
def test_every_element_at_stride_2(B, ctx, oracle, cfg, shape):
    """Odd and even maps: the last row or column of an even one has no second tap below or beside it, and an odd one no odd pixels."""
    if cfg in (47, 49) and shape[1] <= 4 and shape[0] > 32:
        pytest.skip("rows of too many images for its LDS")
    B.pc_set_plan_override(ctx, cfg, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_MFMA, ("direct2", cfg))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("cfg", [47, 48, 49])
@pytest.mark.parametrize("dims", [(20, 56, 56, 104, 200), (48, 33, 31, 32, 264)])
def test_several_tiles_per_workgroup_at_stride_2(B, ctx, cfg, dims):
    """The loads run on from tile to tile: against a kernel of the other family; see test_more_tiles_than_workgroups."""
    import torch
    from tests._harness import Case, GpuLayer
    layer = I.Layer(*dims, 2)
    g = GpuLayer(B, ctx, Case(layer, "bf16", 8, I.kept_per_filter(0.3, layer.C), tag=("direct2", "tiles")))
    try:
        out = []
        for code in (cfg, 30):
            B.pc_set_plan_override(ctx, code, 0)
            for fn in (B.pc_conv_fwd, B.pc_conv_fwd_relu):
                y = torch.full((layer.N, layer.Ho, layer.Wo, layer.F), float("nan"), dtype=torch.bfloat16, device="cuda")
                fn(ctx, g.desc, g.pk, g.x, y)
                out.append(y.double())
        assert torch.equal(out[1], torch.where(out[0] > 0, out[0], torch.zeros_like(out[0])))
        a, b = out[0], out[2]
        assert bool((a - b).abs().le(2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 2.0 ** -12 * b.abs().max()).all())
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        g.close()


@pytest.mark.parametrize("cfg", [37, 38])
@pytest.mark.parametrize("dims", [(20, 56, 56, 200, 104), (48, 33, 31, 264, 32), (64, 35, 29, 136, 72)])
def test_several_tiles_per_workgroup_at_stride_2_backward(B, ctx, cfg, dims):
    """432 to 1020 tiles of 4, 1 and 3 chunks on 256 workgroups: the three buffers run on from tile to tile at every offset. Against a kernel of
    the other family; see test_more_tiles_than_workgroups."""
    import torch
    from tests._harness import Case, GpuLayer
    layer = I.Layer(*dims, 2)
    g = GpuLayer(B, ctx, Case(layer, "bf16", 8, I.kept_per_filter(0.3, layer.C), tag=("direct2", "back")))
    try:
        out = []
        for code, name in ((cfg, "pc_mfma_conv_solo_kernel<2"), (33, "pc_mfma_conv_mc_kernel")):
            B.pc_set_plan_override(ctx, code, 0)
            dx = torch.full((layer.N, layer.H, layer.W, layer.C), float("nan"), dtype=torch.bfloat16, device="cuda")
            B.pc_conv_bwd_data(ctx, g.desc, g.pk, g.dy, dx)
            assert B.pc_last_kernel(ctx).startswith(name)
            out.append(dx.double())
        a, b = out
        assert bool((a - b).abs().le(2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 2.0 ** -12 * b.abs().max()).all())
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        g.close()


@pytest.mark.parametrize("cfg", [40, 41, 42, 43, 45, 46, 50])
@pytest.mark.parametrize("dims", [(70, 4, 4), (75, 2, 3), (90, 1, 5), (40, 1, 1)])
def test_many_small_images(B, ctx, oracle, cfg, dims):
    """More images than a tile has rows, down to one row each: the rows above and below most rows of a tile, or one of them, are zeros."""
    B.pc_set_plan_override(ctx, cfg, 0)
    try:
        run_case(B, ctx, oracle, dims + (56 if cfg == 50 else 72, 64, 1), "bf16", 8, 0.3, B.PC_VARIANT_MFMA, ("direct", cfg))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("cfg", [-1, 40, 41, 42, 43, 45, 46])
@pytest.mark.parametrize("dims", [(16, 56, 56, 64, 128), (32, 56, 56, 40, 256), (24, 57, 50, 32, 192)])
def test_more_tiles_than_workgroups(B, ctx, cfg, dims):
    """Layers of the size it is for, whose tiles fill one to three rounds and leave some: against a kernel of the other family,
    which adds in another order."""
    import torch
    from tests._harness import Case, GpuLayer
    layer = I.Layer(*dims, 1)
    g = GpuLayer(B, ctx, Case(layer, "bf16", 8, I.kept_per_filter(0.3, layer.C), tag=("direct", "auto")))
    try:
        out = []
        for code in (cfg, 20):
            B.pc_set_plan_override(ctx, code, 0)
            y = torch.full((layer.N, layer.Ho, layer.Wo, layer.F), float("nan"), dtype=torch.bfloat16, device="cuda")
            B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, y)
            out.append((B.pc_last_kernel(ctx), y.double()))
        assert ("pc_mfma_conv_dma_kernel" if cfg in (40, 41, 42) else "pc_mfma_conv_solo_kernel" if cfg > 0 else "pc_mfma_conv_") in out[0][0]
        assert "pc_mfma_conv_ks_kernel" in out[1][0]
        # two roundings to bf16 of sums that differ in the order of float32 additions: at most one unit in the last place apart
        a, b = out[0][1], out[1][1]
        assert bool((a - b).abs().le(2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 2.0 ** -12 * b.abs().max()).all())
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        g.close()


@pytest.mark.parametrize("cfg", [40, 41, 42, 43, 45, 46])
@pytest.mark.parametrize("dims", [(6, 10, 9, 128, 160), (2, 33, 70, 24, 72), (9, 96, 95, 16, 200)])
def test_fused_relu(B, ctx, cfg, dims):
    """Bit-identical to the plain launch followed by the step."""
    import torch
    from tests._harness import Case, GpuLayer
    L = I.Layer(*dims, 1)
    g = GpuLayer(B, ctx, Case(L, "bf16", 8, I.kept_per_filter(0.3, L.C), tag=("direct_relu", cfg)))
    try:
        B.pc_set_plan_override(ctx, cfg, 0)
        y = torch.empty((L.N, L.Ho, L.Wo, L.F), dtype=torch.bfloat16, device="cuda")
        a, dx = torch.full_like(y, float("nan")), torch.empty((L.N, L.H, L.W, L.C), dtype=torch.bfloat16, device="cuda")
        dz = torch.full_like(dx, float("nan"))
        B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, y)
        B.pc_conv_fwd_relu(ctx, g.desc, g.pk, g.x, a)
        B.pc_conv_bwd_data(ctx, g.desc, g.pk, g.dy, dx)
        B.pc_conv_bwd_data_relu(ctx, g.desc, g.pk, g.dy, g.x, dz)
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.int16), torch.where(y > 0, y, torch.zeros_like(y)).view(torch.int16))
        assert torch.equal(dz.view(torch.int16), torch.where(g.x > 0, dx, torch.zeros_like(dx)).view(torch.int16))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        g.close()


@pytest.mark.parametrize("off", [1, 4])
@pytest.mark.parametrize("shape", [(9, 38, 41, 56, 64, 1), (13, 33, 47, 40, 72, 1), (33, 7, 7, 136, 200, 1), (20, 14, 14, 64, 128, 2), (5, 33, 31, 40, 72, 2)])
def test_addresses_that_are_no_multiple_of_16(B, ctx, oracle, shape, off):
    """Tensors that start 2 and 8 bytes past one: the kernels that load through registers take them, with the same bound."""
    import numpy as np
    import torch
    from tests._harness import TOL_L2, TOL_L2_DW, Case, GpuLayer, Guarded, assert_close, from_dev_f32, oracle_masks
    L = I.Layer(*shape)
    case = Case(L, "bf16", 8, I.kept_per_filter(0.3, L.C), tag=("address", shape))
    g = GpuLayer(B, ctx, case)

    def moved(t):
        b = torch.empty((t.numel() + 8,), dtype=t.dtype, device="cuda")
        b[off:off + t.numel()] = t.reshape(-1)
        return b, b.data_ptr() + 2 * off

    try:
        pid, kp, M, Wm = oracle_masks(oracle, case)
        (xb, x), (db, dy) = moved(g.x), moved(g.dy)
        y, dx, dz, dw = Guarded(g.dy.numel() + 8, g.tdt), Guarded(g.x.numel() + 8, g.tdt), Guarded(g.x.numel() + 8, g.tdt), Guarded(g.nnzk * 4, torch.float32)
        B.pc_conv_fwd(ctx, g.desc, g.pk, x, y.ptr + 2 * off)
        B.pc_conv_bwd_data(ctx, g.desc, g.pk, dy, dx.ptr + 2 * off)
        B.pc_conv_bwd_data_relu(ctx, g.desc, g.pk, dy, x, dz.ptr + 2 * off)
        B.pc_conv_bwd_weight(ctx, g.desc, g.pk, x, dy, dw.ptr)
        many = Guarded(g.nnzk * 4, torch.float32)
        B.pc_conv_bwd_weight_batch(ctx, [g.desc], [g.pk], [x], [dy], [many.ptr])
        torch.cuda.synchronize()
        for b in (y, dx, dz, dw, many):
            assert b.margins_intact()
        cut = lambda b, t: from_dev_f32(b.body[off:off + t.numel()]).reshape(t.shape)
        assert_close(cut(y, g.dy), oracle.conv_fwd(case.x, Wm, L.stride), oracle.conv_fwd(np.abs(case.x), np.abs(Wm), L.stride), "bf16", TOL_L2["bf16"], "forward")
        want = oracle.conv_bwd_data(case.dy, Wm, case.x.shape, L.stride)
        assert_close(cut(dx, g.x), want, oracle.conv_bwd_data(np.abs(case.dy), np.abs(Wm), case.x.shape, L.stride), "bf16", TOL_L2["bf16"], "backward-data")
        assert np.array_equal(cut(dz, g.x), np.where(case.x > 0, cut(dx, g.x), 0.0))
        ref = oracle.conv_bwd_weight(case.x, case.dy, M, L.stride), oracle.conv_bwd_weight(np.abs(case.x), np.abs(case.dy), M, L.stride)
        assert_close(g.scatter(dw.body), *ref, "f32", TOL_L2_DW, "backward-weight")
        assert_close(g.scatter(many.body), *ref, "f32", TOL_L2_DW, "backward-weight, several layers")
    finally:
        g.close()


@pytest.mark.parametrize("code", [40, 41, 42])
@pytest.mark.parametrize("shape", [(2, 30, 37, 40, 8, 1), (3, 17, 66, 32, 24, 1), (1, 65, 9, 72, 32, 1), (6, 16, 15, 8, 16, 1), (9, 64, 70, 16, 32, 1)])
def test_up_to_32_output_channels(B, ctx, oracle, code, shape):
    """Half of a tile's 64 channels, forward and, with the channels exchanged, backward-data: filters that do not fill 32, chunks that end early,
    tiles across images, rows and columns past the map, rounds and their pieces; with the fused ReLU and its mask."""
    import torch
    from tests._harness import Case, GpuLayer, Guarded
    N, H, W, C, F, stride = shape
    for c, f in ((C, F), (F, C)):
        B.pc_set_plan_override(ctx, code, 0)
        L = I.Layer(N, H, W, c, f, stride)
        g = None
        try:
            run_case(B, ctx, oracle, (N, H, W, c, f, stride), "bf16", 8, 0.4, B.PC_VARIANT_MFMA, "narrow")
            g = GpuLayer(B, ctx, Case(L, "bf16", 8, I.kept_per_filter(0.4, c), tag=("narrow", c, f)))
            fwd = f <= 32
            n = L.N * L.H * L.W * (f if fwd else c)
            z, a = (Guarded(n, torch.bfloat16) for _ in range(2))
            (B.pc_conv_fwd if fwd else B.pc_conv_bwd_data)(ctx, g.desc, g.pk, g.x if fwd else g.dy, z.ptr)
            assert B.pc_last_kernel(ctx).startswith("pc_mfma_conv_dma_kernel<") and B.pc_last_kernel(ctx).endswith(", 2>")
            if fwd:
                B.pc_conv_fwd_relu(ctx, g.desc, g.pk, g.x, a.ptr)
                keep = z.body > 0
            else:
                B.pc_conv_bwd_data_relu(ctx, g.desc, g.pk, g.dy, g.x, a.ptr)
                keep = g.x.reshape(-1).view(torch.bfloat16) > 0
            torch.cuda.synchronize()
            assert z.margins_intact() and a.margins_intact()
            assert torch.equal(a.body.view(torch.int16), torch.where(keep, z.body, torch.zeros_like(z.body)).view(torch.int16))
        finally:
            B.pc_set_plan_override(ctx, -1, 0)
            if g is not None:
                g.close()
