"""The weight gradient of a layer with few pixels in one launch (override code 55; split_k picks its tile), element by element against the
oracle: maps of one row and one column, tiles cut by the channel counts, several chunks of pixels, steps that do not divide among the
wavefronts; and that it needs no scratch."""
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
    (1, 1, 1, 8, 8, 1),           # one pixel
    (3, 1, 5, 24, 40, 1),         # maps of one row and of one column
    (5, 7, 1, 40, 24, 1),
    (9, 2, 2, 72, 136, 1),        # more cells than pixels
    (1, 14, 14, 264, 96, 1),
    (2, 33, 31, 16, 32, 1),       # one chunk of one tile, two of another
    (4, 40, 39, 56, 48, 1),       # several chunks, the last not full
    (1, 5, 200, 32, 16, 1)]       # a long row


@pytest.mark.parametrize("tile", [0, 1, 2, 3])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_element(B, ctx, oracle, tile, shape):
    B.pc_set_plan_override(ctx, 55, tile)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.4, B.PC_VARIANT_MFMA, ("few_wgrad", tile))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("dims", [(2, 9, 8, 64, 96), (30, 6, 7, 256, 128)])
def test_same_bits_without_scratch(B, dims):
    """Under capture on a context that has no scratch, and by the entry that allocates nothing."""
    import torch
    from tests._harness import Case, GpuLayer
    stream = torch.cuda.Stream()
    c = B.pc_create(0, stream.cuda_stream)
    layer = I.Layer(*dims, 1)
    try:
        with torch.cuda.stream(stream):
            g = GpuLayer(B, c, Case(layer, "bf16", 8, I.kept_per_filter(0.5, layer.C), tag=("few", "capture")))
            want, got, other = (torch.full((g.nnzk, 4), float("nan"), device="cuda") for _ in range(3))
            B.pc_conv_bwd_weight(c, g.desc, g.pk, g.x, g.dy, want)
            assert B.pc_last_kernel(c).startswith("pc_mfma_wgrad_dma_few_kernel")
            B.pc_conv_bwd_weight_noalloc(c, g.desc, g.pk, g.x, g.dy, other)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            B.pc_conv_bwd_weight(c, g.desc, g.pk, g.x, g.dy, got)
        for _ in range(3):
            with torch.cuda.stream(stream):
                got.fill_(float("nan"))
                graph.replay()            # (on this stream: behind the fill)
            torch.cuda.synchronize()
            assert torch.equal(got, want) and torch.equal(other, want)
        g.close()
    finally:
        B.pc_destroy(c)
