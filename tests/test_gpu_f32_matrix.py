"""The float32 matrix-core kernels at the edges of their tiles: one pixel, maps narrower than a strip and strips that do
not divide the map, tiles that cross images, channel counts around 8, 32 and 64 and rows that are no whole 16 bytes, the
first layer's (tap, channel) columns, stride 2 on odd maps; all three passes against the oracle element by element."""
import pytest

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
    (1, 1, 1, 3, 5, 1), (1, 1, 1, 8, 32, 2), (9, 1, 1, 33, 64, 1), (2, 5, 67, 33, 36, 1), (3, 7, 7, 40, 130, 2), (5, 9, 2, 4, 97, 1),
    (1, 3, 200, 8, 32, 1), (2, 6, 5, 64, 64, 2), (17, 3, 3, 72, 24, 1), (2, 31, 29, 2, 48, 1), (4, 13, 13, 1, 70, 2), (3, 8, 8, 256, 31, 1),
    (40, 14, 14, 65, 68, 1), (6, 4, 33, 24, 200, 2)])
def test_edges(B, ctx, oracle, shape):
    run_case(B, ctx, oracle, shape, "f32", 8, 0.4, B.PC_VARIANT_AUTO, "f32_matrix")
    assert B.pc_last_kernel(ctx).startswith("pc_f32_wgrad_kernel")


@pytest.mark.parametrize("shape", [(2, 9, 9, 24, 40, 1), (3, 8, 7, 12, 33, 2)])
def test_gather_kernels_still_take_float32(B, ctx, oracle, shape):
    run_case(B, ctx, oracle, shape, "f32", 8, 0.4, B.PC_VARIANT_VALU, "f32_gather")
    assert B.pc_last_kernel(ctx).startswith("pc_wgrad_valu_kernel")


@pytest.mark.parametrize("waves,shape", [
    ("1, 1", (1, 29, 3, 100, 40, 1)), ("1, 1", (1, 4, 22, 24, 66, 1)), ("1, 1", (8, 45, 2, 130, 64, 1)), ("1, 2", (6, 2, 19, 100, 64, 1)), ("1, 2", (1, 13, 4, 40, 130, 1)),
    ("1, 2", (4, 6, 22, 40, 33, 1)), ("2, 1", (1, 3, 34, 24, 40, 2)), ("2, 1", (1, 18, 12, 130, 130, 2)), ("2, 1", (11, 8, 49, 33, 40, 1)), ("2, 1", (3, 30, 31, 2, 50, 2)),
    ("2, 2", (1, 3, 5, 8, 66, 2)), ("2, 2", (2, 12, 1, 33, 66, 1))])
def test_wavefronts_that_share_pixels(B, ctx, oracle, waves, shape):
    """Weight gradients whose wavefronts add their sums in LDS: two and four of them, rows of quads and not, the (tap, channel) columns of a first layer."""
    run_case(B, ctx, oracle, shape, "f32", 8, 0.4, B.PC_VARIANT_AUTO, "f32_shared")
    assert B.pc_last_kernel(ctx).startswith("pc_f32_wgrad_kernel<%s, " % waves)


@pytest.mark.parametrize("kernel,shape", [
    ("2, 2, 1, 2", (6, 55, 55, 8, 40, 1)), ("2, 2, 1, 2", (2, 94, 97, 3, 48, 1)), ("4, 1, 1, 2", (11, 33, 32, 16, 96, 1)), ("4, 1, 1, 2", (2, 111, 113, 3, 136, 2)),
    ("1, 4, 1, 2", (43, 30, 32, 8, 24, 1)), ("1, 4, 1, 2", (12, 60, 58, 3, 24, 1)), ("2, 2, 1, 1", (10, 34, 32, 8, 24, 1)), ("4, 1, 1, 1", (15, 6, 7, 32, 464, 1)),
    ("4, 1, 1, 1", (88, 8, 10, 3, 48, 1)), ("1, 4, 1, 1", (1, 138, 139, 32, 24, 1)), ("1, 4, 1, 1", (117, 27, 25, 3, 24, 1))])
def test_three_parts(B, ctx, oracle, kernel, shape):
    """Tiles of 32, operands split in three: every shape of workgroup, half a fragment of 16 channels, rows that are no whole quads. Next to the
    element-wise bound of float32: the error over the whole tensor is that of sums rounded after sixteen products, not after two."""
    import numpy as np
    from paper_2011_10170_amd import inputs as I
    from tests._harness import Case, GpuLayer, oracle_masks
    run_case(B, ctx, oracle, shape, "f32", 8, 0.4, B.PC_VARIANT_AUTO, "f32_parts")
    L = I.Layer(*shape)
    case = Case(L, "f32", 8, I.kept_per_filter(0.4, L.C), tag=("parts", shape))
    Wm = oracle_masks(oracle, case)[3]
    g = GpuLayer(B, ctx, case)
    try:
        y = g.fwd()
        assert B.pc_last_kernel(ctx).startswith("pc_f32_conv_kernel<32, %s, " % kernel)
    finally:
        g.close()
    ref = oracle.conv_fwd(case.x, Wm, L.stride)
    # n additions that each round the running sum by at most 2^-24 of it (0.58 of that in the mean square) and of which the sum
    # has half its final square on average, and the final rounding; n = the groups of 16 channels of every tap, twice for the hardware's own halves
    n = 9 * -(-L.C // 16) * 2
    bound = 2.0 ** -24 * (1.0 + 0.58 * np.sqrt(n / 2.0))
    rel = float(np.linalg.norm(y.astype(np.float64) - ref) / np.linalg.norm(ref))
    print("error over the tensor: %.2e, bound %.2e" % (rel, bound))
    assert rel <= bound, (rel, bound)
