"""Float32 layers far from 1: operands down to float32's subnormals and sums up to its largest values keep float32's 24 bits, whichever kernel
the layer's size goes to. Every element of the three passes against the oracle; no result itself is subnormal."""
import numpy as np
import pytest

from paper_2011_10170_amd import inputs as I
from tests._harness import Case, GpuLayer, TOL_L2, TOL_L2_DW, assert_close, oracle_masks, to_dev

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


# x, the weights and dy are scaled by these powers of two: each small beside two that are large, 2^-140 subnormal with 9 bits and less. (Products
# of the large ones are beyond 2^96, where the scaled sums overflow and the kept taps are multiplied again.)
SCALES = [tuple(small if i == k else 45 for i in range(3)) for small in (-112, -120, -130, -140) for k in range(3)]


# tiles of 16 and of 32 (both widths of a wavefront, the last round in parts, the reduction along four wavefronts, the parity classes of
# stride 2); weight gradients whose wavefronts share pixels and do not, and of the first layer's (tap, channel) columns
@pytest.mark.parametrize("shape", [(2, 11, 13, 48, 24, 1), (12, 28, 28, 64, 128, 1), (10, 34, 32, 8, 24, 1), (3, 7, 7, 40, 130, 2), (9, 56, 57, 24, 100, 2), (2, 31, 29, 3, 48, 1)])
def test_three_passes(B, ctx, oracle, shape):
    L = I.Layer(*shape)
    case = Case(L, "f32", 8, I.kept_per_filter(0.3, L.C), tag=("scales", shape))
    pid, kp, M, _ = oracle_masks(oracle, case)
    sf, sc = oracle.compact_order(pid, kp, case.P)
    g = GpuLayer(B, ctx, case)
    try:
        for ex, ew, ed in SCALES:
            # (half of the images stay 2^8 times larger: small and less small operands meet in a tile)
            step = np.where(np.arange(L.N) % 2, 0, 8).reshape(-1, 1, 1, 1)
            x, dy, W = (np.ldexp(v, e).astype(np.float32) for v, e in ((case.x, ex + step), (case.dy, ed + step), (case.W, ew)))
            Wm = oracle.apply_mask(W, M)
            g.x, g.dy = to_dev(x), to_dev(dy)
            B.pc_update_values(ctx, g.pk, to_dev(W))
            what = "%s x 2^%d, W 2^%d, dy 2^%d: " % (shape, ex, ew, ed)
            assert_close(g.fwd(), oracle.conv_fwd(x, Wm, L.stride), oracle.conv_fwd(np.abs(x), np.abs(Wm), L.stride), "f32", TOL_L2["f32"], what + "fwd")
            assert_close(g.bwd_data(), oracle.conv_bwd_data(dy, Wm, x.shape, L.stride), oracle.conv_bwd_data(np.abs(dy), np.abs(Wm), x.shape, L.stride), "f32",
                         TOL_L2["f32"], what + "bwd_data")
            ref, mag = (oracle.gather_compact(oracle.conv_bwd_weight(p, q, M, L.stride), pid, case.lib, sf, sc) for p, q in ((x, dy), (np.abs(x), np.abs(dy))))
            assert_close(g.bwd_weight()[0], ref, mag, "f32", TOL_L2_DW, what + "bwd_weight")
    finally:
        g.close()
