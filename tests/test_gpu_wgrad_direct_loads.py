"""Backward-weight from NHWC rows in LDS (override code 44), element by element against the oracle: rows that run across images,
rows and columns past the map, partial tiles of filters and channels, both strides, one split and many; and several layers in one
call, some of which the kernel does not take."""
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


@pytest.mark.parametrize("shape", [
    (1, 1, 1, 8, 8, 1), (40, 1, 2, 8, 8, 1), (3, 2, 3, 8, 16, 1), (70, 4, 4, 64, 64, 1), (3, 8, 8, 72, 64, 1), (9, 7, 7, 136, 200, 1),
    (1, 33, 47, 40, 72, 1), (2, 64, 31, 8, 8, 1), (5, 31, 15, 64, 24, 1), (12, 32, 32, 64, 128, 1), (1, 95, 9, 16, 264, 1),
    (1, 1, 1, 8, 8, 2), (33, 2, 3, 8, 16, 2), (70, 4, 4, 64, 64, 2), (9, 7, 7, 136, 200, 2), (3, 14, 14, 24, 72, 2), (1, 33, 47, 40, 72, 2),
    (2, 64, 47, 136, 16, 2), (5, 15, 16, 64, 128, 2)])
def test_backward_weight(B, ctx, oracle, shape):
    B.pc_set_plan_override(ctx, 44, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_MFMA, ("rows", shape))
        assert B.pc_last_kernel(ctx).startswith("pc_mfma_wgrad_dma_kernel")
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("waves", [1, 2, 3])
@pytest.mark.parametrize("shape", [
    (1, 1, 1, 8, 8, 1), (40, 1, 2, 8, 8, 1), (3, 5, 3, 40, 32, 1), (9, 7, 7, 32, 200, 1), (1, 33, 47, 40, 72, 1), (5, 31, 15, 64, 24, 1), (4, 64, 40, 32, 32, 1),
    (1, 1, 1, 8, 8, 2), (33, 2, 3, 8, 16, 2), (9, 7, 7, 136, 32, 2), (1, 33, 47, 40, 72, 2), (2, 64, 47, 24, 16, 2)])
def test_wavefronts_that_share_pixels(B, ctx, oracle, waves, shape):
    """Tiles of 32 filters or channels (split_k names the arrangement): the wavefronts' sums are added in LDS."""
    B.pc_set_plan_override(ctx, 44, waves)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.4, B.PC_VARIANT_MFMA, ("rows", shape))
        assert B.pc_last_kernel(ctx) == "pc_mfma_wgrad_dma_kernel<%d, %s>" % (shape[5], ("1, 2", "2, 1", "1, 1")[waves - 1])
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


SMALL = [(6, 14, 14, 64, 72, 1), (6, 14, 14, 3, 64, 1), (6, 27, 28, 40, 24, 2), (6, 7, 7, 136, 64, 1)]


@pytest.mark.parametrize("code", [44, -1])
@pytest.mark.parametrize("dims", [
    SMALL, SMALL + [(6, 9, 9, 24, 12, 1)],
    [(32, 56, 56, 64, 128, 1), (32, 56, 56, 128, 128, 1), (32, 57, 55, 72, 128, 2), (32, 28, 28, 128, 256, 1), (32, 28, 28, 256, 200, 1)]])
def test_several_layers(B, ctx, code, dims):
    """Against the single calls of the wave-specialised kernel (where it takes a layer), which add in another order: the difference of two
    float32 sums of n terms each, all of them pixels' products."""
    import torch
    from tests._harness import Case, GpuLayer
    if code == 44 and any(s[4] % 8 for s in dims):
        pytest.skip("a forced kernel refuses a layer that neither it nor the wave-specialised one takes")
    gs = [GpuLayer(B, ctx, Case(I.Layer(*s), "bf16", 8, I.kept_per_filter(0.3, s[3]), tag=("rows", s))) for s in dims]
    try:
        want = []
        B.pc_set_plan_override(ctx, 11, 0)
        for g in gs:
            try:
                w = torch.zeros((g.nnzk, 4), device="cuda")
                B.pc_conv_bwd_weight(ctx, g.desc, g.pk, g.x, g.dy, w)
            except B.PcError:
                B.pc_set_plan_override(ctx, 10, 0)
                B.pc_conv_bwd_weight(ctx, g.desc, g.pk, g.x, g.dy, w)
                B.pc_set_plan_override(ctx, 11, 0)
            want.append(w)
        B.pc_set_plan_override(ctx, code, 0)
        got = [torch.full((g.nnzk, 4), float("nan"), device="cuda") for g in gs]
        B.pc_conv_bwd_weight_batch(ctx, [g.desc for g in gs], [g.pk for g in gs], [g.x for g in gs], [g.dy for g in gs], got)
        torch.cuda.synchronize()
        for a, b, s in zip(got, want, dims):
            # every chain of additions loses at most 2^-24 of its running sum a step and is combined pairwise; the sums' terms are of both
            # signs, so a running sum stays within a few times the root of the number of pixels
            n = s[0] * ((s[1] - 1) // s[5] + 1) * ((s[2] - 1) // s[5] + 1)
            bound = 2.0 ** -24 * 64 * np.sqrt(n)
            assert bool(((a - b).abs() <= bound + 2.0 ** -18 * b.abs()).all()), s
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        for g in gs:
            g.close()


@pytest.mark.parametrize("code", [44, 11, -1])
def test_several_layers_against_the_oracle(B, ctx, oracle, code):
    """One call for layers of both strides, whole images and strips of them, and channels that fill no tile; at code 44 also one that is left to the
    other kernel (3 channels)."""
    import torch
    from tests._harness import TOL_L2_DW, Case, GpuLayer, Guarded, assert_close, oracle_masks
    dims = SMALL + [(33, 8, 8, 64, 136, 1), (3, 15, 16, 72, 128, 2)]
    gs = [GpuLayer(B, ctx, Case(I.Layer(*s), "bf16", 8, I.kept_per_filter(0.3, s[3]), tag=("group", s))) for s in dims]
    try:
        B.pc_set_plan_override(ctx, code, 0)
        out = [Guarded(g.nnzk * 4, torch.float32) for g in gs]
        B.pc_conv_bwd_weight_batch(ctx, [g.desc for g in gs], [g.pk for g in gs], [g.x for g in gs], [g.dy for g in gs], [b.ptr for b in out])
        torch.cuda.synchronize()
        for g, b, s in zip(gs, out, dims):
            assert b.margins_intact()
            c = g.case
            _, _, M, _ = oracle_masks(oracle, c)
            assert_close(g.scatter(b.body), oracle.conv_bwd_weight(c.x, c.dy, M, s[5]), oracle.conv_bwd_weight(np.abs(c.x), np.abs(c.dy), M, s[5]), "f32", TOL_L2_DW,
                         "%s" % (s,))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        for g in gs:
            g.close()


def test_capture_without_room_for_the_partial_planes(B):
    """A call whose partial planes would need more scratch than there is, under stream capture: the kernel with fewer planes takes it."""
    import torch
    from tests._harness import Case, GpuLayer
    stream = torch.cuda.Stream()
    c = B.pc_create(0, stream.cuda_stream)
    layer = I.Layer(64, 56, 56, 128, 128, 2)
    try:
        with torch.cuda.stream(stream):
            g = GpuLayer(B, c, Case(layer, "bf16", 8, I.kept_per_filter(0.5, layer.C), tag=("rows", "capture")))
            want, got = (torch.zeros((g.nnzk, 4), device="cuda") for _ in range(2))
            B.pc_set_plan_override(c, 11, 0)
            B.pc_conv_bwd_weight(c, g.desc, g.pk, g.x, g.dy, want)
            B.pc_set_plan_override(c, -1, 0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.pc_conv_bwd_weight(c, g.desc, g.pk, g.x, g.dy, got)
        assert B.pc_last_kernel(c).startswith("pc_mfma_wgrad_ws_kernel")
        for _ in range(3):
            with torch.cuda.stream(stream):
                got.fill_(float("nan"))
                graph.replay()            # (on this stream: behind the fill)
            torch.cuda.synchronize()
            assert torch.equal(got, want)
        with torch.cuda.stream(stream):
            B.pc_conv_bwd_weight(c, g.desc, g.pk, g.x, g.dy, got)
        assert B.pc_last_kernel(c).startswith("pc_mfma_wgrad_dma_kernel")
        torch.cuda.synchronize()
        g.close()
    finally:
        B.pc_destroy(c)
