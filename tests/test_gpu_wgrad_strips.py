"""Backward-weight of batches that are no multiple of 8: the images are cut into strips of rows so that the groups of 8 fill.
Odd maps that the strips do not divide, both strides, maps with fewer rows than strips, the first layer's form, several
layers in one call; element by element against the oracle."""
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
    (1, 1, 1, 8, 8, 1), (1, 3, 40, 16, 24, 1), (1, 37, 41, 40, 72, 1), (2, 29, 17, 72, 40, 1), (3, 31, 30, 24, 136, 1),
    (5, 13, 50, 64, 64, 1), (7, 9, 9, 80, 16, 1), (9, 21, 7, 32, 96, 1), (13, 33, 47, 40, 72, 1), (1, 45, 39, 24, 56, 2),
    (3, 27, 28, 40, 24, 2), (6, 15, 15, 64, 72, 2), (1, 57, 61, 3, 64, 1), (5, 20, 33, 3, 24, 2)])
def test_backward_weight_of_short_batches(B, ctx, oracle, shape):
    run_case(B, ctx, oracle, shape, "bf16", 8, 0.3, B.PC_VARIANT_AUTO, ("strips", shape))
