"""Layers ranked as a whole by two launches, and packs written by one: at the edges of the sizes that take them, with ties at the cut,
scores that share one bin and scores below every bin. Bit-exact against the oracle, and against the order of the compact kernels."""
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


# 16385 kernels: the first size; 65536 kernels: the last; one past it
@pytest.mark.parametrize("values", ["normal", "few", "equal", "tiny"])
@pytest.mark.parametrize("shape", [(113, 145), (199, 217), (64, 1024), (511, 127), (223, 294)])
def test_layer_ranked_as_a_whole(B, ctx, oracle, shape, values):
    import torch
    F, C = shape
    lib = I.make_library(8)
    rng = np.random.default_rng(F * 7 + C)
    if values == "few":                     # many scores equal to the threshold, in every bin
        Wn, Gn = (rng.integers(-2, 3, size=(F, C, 9)).astype(np.float32) * 0.5 for _ in range(2))
    elif values == "equal":                 # one score, taken by index
        Wn = Gn = np.ones((F, C, 9), np.float32)
    else:
        Wn, Gn = (rng.standard_normal((F, C, 9)).astype(np.float32) for _ in range(2))
        if values == "tiny":                # scores are subnormal or zero
            Wn = Wn * np.float32(1e-21)
    L = F * C
    Wd, Gd = to_dev(Wn), to_dev(Gn)
    for n_keep in (1, L // 3, L - 1):
        pid, keep = oracle.select(Wn, Gn, lib, n_keep, keep_mode=1, score_mode=0)
        gp, gk = (torch.full((F, C), 255, dtype=torch.uint8, device="cuda") for _ in range(2))
        B.pc_pattern_select(ctx, Wd, Gd, F, C, lib, 1, n_keep, 0, gp, gk)
        torch.cuda.synchronize()
        assert np.array_equal(gp.cpu().numpy(), pid), n_keep
        assert np.array_equal(gk.cpu().numpy(), keep), n_keep


# one launch: rows of up to 512 kernels and up to 131072 in all, masks on 16-byte boundaries
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,offset", [((1, 1), 0), ((33, 31), 0), ((64, 72), 0), ((256, 512), 0), ((127, 513), 0), ((257, 511), 0),
                                          ((256, 256), 0), ((256, 256), 1), ((3, 129), 0)])
def test_pack_order(B, ctx, shape, offset, dtype):
    import torch
    F, C = shape
    lib = I.make_library(12)
    rng = np.random.default_rng(F * 11 + C)
    W = rng.standard_normal((F, C, 9)).astype(np.float32)
    pid = rng.integers(0, 14, size=(F, C)).astype(np.uint8)      # an id past the pool is no kept kernel
    keep = (rng.random((F, C)) < 0.4).astype(np.uint8) * rng.integers(1, 256, size=(F, C)).astype(np.uint8)

    def place(a):
        buf = torch.zeros(F * C + 16, dtype=torch.uint8, device="cuda")
        buf[offset:offset + F * C] = to_dev(a.reshape(-1))
        return buf[offset:offset + F * C].view(F, C)
    pk = B.pc_pack(ctx, to_dev(W), place(pid), place(keep), F, C, lib, B.PC_F32 if dtype == "f32" else B.PC_BF16)
    order = [(f, p, c) for f in range(F) for p, c in sorted((int(pid[f, c]), c) for c in range(C) if keep[f, c] and pid[f, c] < 12)]
    assert B.pc_packed_info(ctx, pk)[0] == len(order)
    dense = torch.full((F, C, 9), -1.0, device="cuda")
    compact = torch.arange(4 * max(1, len(order)), dtype=torch.float32, device="cuda").view(-1, 4) + 1.0
    B.pc_scatter_dense(ctx, pk, compact, dense)
    want = np.zeros((F, C, 9), np.float32)
    for slot, (f, p, c) in enumerate(order):
        want[f, c, [t for t in range(9) if lib[p] >> t & 1]] = 4 * slot + 1 + np.arange(4)
    assert np.array_equal(dense.cpu().numpy(), want)
    B.pc_unpack_dense(ctx, pk, dense)
    value = W if dtype == "f32" else torch.from_numpy(W).to(torch.bfloat16).float().numpy()
    assert np.array_equal(dense.cpu().numpy(), np.where(want != 0, value, 0))
    B.pc_packed_free(pk)
