"""The matrix-core forward / backward-data kernels with tiles of 32 output channels, and the automatic choice on layers with
few channels on either side (8 to 40: partial chunks of every width, partial row tiles), both strides, element by element
against the oracle."""
import pytest

from tests.test_gpu_parity import WAVE_SPEC, run_case

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


@pytest.mark.parametrize("cfg", [24, 25, 26, 27, 28, 29])
@pytest.mark.parametrize("shape", WAVE_SPEC + [(3, 11, 13, 8, 16, 1), (2, 17, 9, 24, 40, 2)])
def test_tiles_of_32_output_channels(B, ctx, oracle, cfg, shape):
    B.pc_set_plan_override(ctx, cfg, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_MFMA, ("thin_rows", cfg))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("cfg", [30, 31])
@pytest.mark.parametrize("shape", WAVE_SPEC + [(2, 17, 9, 24, 136, 2), (3, 33, 31, 72, 200, 2), (11, 28, 29, 40, 128, 2)])
def test_tiles_of_128_output_channels(B, ctx, oracle, cfg, shape):
    B.pc_set_plan_override(ctx, cfg, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_MFMA, ("two_rows", cfg))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)


@pytest.mark.parametrize("shape", [(1, 5, 4, 8, 8, 1), (9, 33, 31, 8, 200, 1), (40, 66, 65, 16, 24, 1), (3, 40, 37, 24, 16, 2),
                                   (30, 65, 66, 8, 40, 2), (2, 9, 7, 424, 8, 1), (1, 19, 23, 16, 328, 2), (33, 6, 5, 200, 32, 1)])
def test_few_channels_automatic(B, ctx, oracle, shape):
    run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_AUTO, ("few", shape))


@pytest.mark.parametrize("cfg", [32, 33, 34, 35, 36])
@pytest.mark.parametrize("shape", [(1, 1, 1, 8, 8, 2), (2, 2, 3, 40, 24, 2), (3, 9, 8, 24, 72, 2), (5, 33, 31, 72, 40, 2), (2, 64, 47, 136, 16, 2),
                                   (70, 7, 7, 64, 200, 2), (9, 56, 56, 32, 64, 2)])
def test_stride2_backward_data_in_one_pass(B, ctx, oracle, cfg, shape):
    """All four parity classes of a tile from one staged neighbourhood: odd and even extents, one pixel, tiles across images,
    partial channel chunks and row tiles, more tiles than workgroups."""
    B.pc_set_plan_override(ctx, cfg, 0)
    try:
        run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_MFMA, ("one_pass", cfg))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
