"""First layer of small batches: the forward tile is cut down until every CU has a workgroup. Maps of fewer rows or columns than a
tile, a last tile of one row or column, every filter count; element by element against the oracle."""
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
    (1, 1, 1, 3, 32, 1), (1, 2, 33, 3, 64, 1), (1, 41, 65, 3, 96, 1), (2, 65, 97, 3, 128, 1), (1, 129, 257, 3, 32, 1), (5, 37, 70, 4, 64, 1),
    (9, 33, 129, 1, 64, 1)])
def test_forward_of_few_tiles(B, ctx, oracle, shape):
    run_case(B, ctx, oracle, shape, "bf16", 8, 0.5, B.PC_VARIANT_AUTO, ("first layer", shape))
