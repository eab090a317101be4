"""Float32 tiles of 16 x 16: reduction lengths that end within a 16-channel fragment or within a chunk of 64 or 128, one to 33
output channels, fewer pixels than a tile, rows that no 16-byte load covers, both strides; element by element against the oracle."""
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
    (1, 1, 1, 8, 8, 1), (1, 5, 3, 24, 16, 1), (2, 11, 13, 360, 24, 1), (1, 7, 9, 136, 17, 1), (3, 4, 5, 72, 33, 1), (1, 6, 17, 37, 15, 1),
    (5, 8, 8, 264, 40, 1), (1, 33, 31, 40, 8, 1), (2, 9, 7, 120, 56, 2), (1, 13, 10, 30, 18, 2), (4, 5, 6, 200, 16, 2), (9, 3, 2, 64, 72, 2)])
def test_layers_of_few_tiles(B, ctx, oracle, shape):
    run_case(B, ctx, oracle, shape, "f32", 8, 0.3, B.PC_VARIANT_AUTO, ("small tiles", shape))
