"""Selection at the sizes where its kernels change: rows ranked in the registers of one wavefront or of several, rows and
layers ranked by one workgroup or across workgroups, the last 64 kernels of a row incomplete, scores with ties at the cut;
and unpacking at the edges of the operand tiles. Bit-exact against the oracle."""
import numpy as np
import pytest

from paper_2011_10170_amd import inputs as I
from tests._harness import to_dev

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


# (F, C, keep mode): one row per workgroup up to 512 kernels, one per wavefront from 8 rows per CU, longer rows by a workgroup with
# the keys in LDS, or with the scores in memory; whole layers up to 16384 kernels by one workgroup
SHAPES = [(5, 1, 0), (7, 63, 0), (7, 65, 0), (4, 512, 0), (4, 513, 0), (2, 4097, 0), (1, 16385, 0), (2100, 65, 0), (2060, 3, 0),
          (64, 64, 1), (3, 1366, 1), (128, 128, 1), (113, 146, 1)]


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_selection_at_the_edges(B, ctx, oracle, shape, ties):
    import torch
    F, C, mode = shape
    lib = I.make_library(12)
    if ties:
        rng = np.random.default_rng(F * 7 + C)
        Wn, Gn = (rng.integers(-2, 3, size=(F, C, 9)).astype(np.float32) * 0.5 for _ in range(2))
    else:
        Wn, Gn = I.gen_weights(F, C, I.BASE_SEED, ("edge", shape)), I.gen_weight_grads(F, C, I.BASE_SEED, ("edge", shape))
    L = C if mode == 0 else F * C
    Wd, Gd = to_dev(Wn), to_dev(Gn)
    for grad in (True, False):
        for n_keep in sorted({0, 1, L // 3, L - 1, L}):
            pid, keep = oracle.select(Wn, Gn if grad else None, lib, n_keep, keep_mode=mode, score_mode=0)
            gp, gk = (torch.full((F, C), 255, dtype=torch.uint8, device="cuda") for _ in range(2))
            B.pc_pattern_select(ctx, Wd, Gd if grad else None, F, C, lib, mode, n_keep, 0, gp, gk)
            torch.cuda.synchronize()
            assert np.array_equal(gp.cpu().numpy(), pid), (n_keep, grad)
            assert np.array_equal(gk.cpu().numpy(), keep), (n_keep, grad)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(1, 1), (33, 31), (64, 72), (31, 513), (130, 1030)])
def test_pack_update_and_unpack_at_the_edges(B, ctx, oracle, shape, dtype):
    import torch
    F, C = shape
    lib = I.make_library(16)
    Wn, Gn = I.gen_weights(F, C, I.BASE_SEED, ("pk", shape)), I.gen_weight_grads(F, C, I.BASE_SEED, ("pk", shape))
    W2 = I.gen_weights(F, C, I.BASE_SEED + 1, ("pk", shape))
    pid, keep = oracle.select(Wn, Gn, lib, max(1, C // 3), keep_mode=0, score_mode=0)
    mask = np.zeros((F, C, 9), bool)
    for t in range(9):
        mask[:, :, t] = ((np.asarray(lib, np.uint32)[pid] >> t) & 1).astype(bool) & (keep != 0)
    dt = B.PC_BF16 if dtype == "bf16" else B.PC_F32
    dense = torch.full((F, C, 9), np.nan, dtype=torch.float32, device="cuda")
    pk = B.pc_pack(ctx, to_dev(Wn), to_dev(pid), to_dev(keep), F, C, lib, dt)
    for w in (Wn, W2):
        if w is W2:
            B.pc_update_values(ctx, pk, to_dev(W2))
        B.pc_unpack_dense(ctx, pk, dense)
        want = torch.from_numpy(np.where(mask, w, np.float32(0)))
        if dtype == "bf16":
            want = want.to(torch.bfloat16).to(torch.float32)
        assert torch.equal(dense.cpu(), want)
    # compact order: filter, pattern id, channel
    n = B.pc_packed_info(ctx, pk)[0]
    comp = torch.arange(4 * n, dtype=torch.float32, device="cuda") + 1
    B.pc_scatter_dense(ctx, pk, comp, dense)
    order = [(f, int(pid[f, c]), c) for f in range(F) for c in range(C) if keep[f, c]]
    want = np.zeros((F, C, 9), np.float32)
    for slot, (f, p, c) in enumerate(sorted(order)):
        want[f, c, [t for t in range(9) if lib[p] >> t & 1]] = 4 * slot + 1 + np.arange(4)
    assert n == len(order) and np.array_equal(dense.cpu().numpy(), want)
    B.pc_packed_free(pk)
