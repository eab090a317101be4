"""Float32 launches whose last, partly filled round runs in parts of 32 x 32: each tile shape, tiles that end past the pixels or
past the output channels, tiles across images and strips, both strides, one round and several; element by element against the
oracle."""
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
    (9, 25, 80, 24, 128, 1), (6, 35, 68, 30, 136, 1), (6, 77, 85, 17, 64, 1), (8, 47, 44, 64, 100, 1), (8, 80, 78, 33, 32, 1),
    (7, 58, 46, 24, 34, 1), (5, 72, 46, 17, 128, 1), (9, 112, 110, 24, 100, 2)])
def test_last_round_in_parts(B, ctx, oracle, shape):
    run_case(B, ctx, oracle, shape, "f32", 8, 0.3, B.PC_VARIANT_AUTO, ("last round", shape))
