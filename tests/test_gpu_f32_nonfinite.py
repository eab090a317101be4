"""Infinite and NaN elements in float32 layers: a pruned tap and the zeros around the maps take no part in a sum, although the matrix
instructions multiply them. Every element of the three passes against the oracle (kept taps inside the maps only): the same
infinities and NaN at the same places, everything else within the bound of finite inputs. One shape per kind of kernel."""
import numpy as np
import pytest

from paper_2011_10170_amd import inputs as I
from tests._harness import Case, GpuLayer, TOL_L2, TOL_L2_DW, assert_close, oracle_masks, to_dev

pytestmark = pytest.mark.gpu

BAD = (np.inf, -np.inf, np.nan)


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


def spoiled(t, rng):
    """t with non-finite elements in the first and the last pixel (corners of a map) and at random places."""
    t = t.copy()
    flat = t.reshape(-1, t.shape[-1])
    at = [0, len(flat) - 1] + list(rng.integers(0, len(flat), size=4))
    for i, p in enumerate(at):
        flat[p, rng.integers(0, t.shape[-1])] = BAD[i % 3]
    return t


def check(got, ref, mag, l2, what):
    assert np.array_equal(np.isnan(got), np.isnan(ref)), (what, "NaN")
    for inf in (np.inf, -np.inf):
        assert np.array_equal(got == inf, ref == inf), (what, inf)
    ok = np.isfinite(ref)
    print("  %s: %d of %d elements not finite" % (what, (~ok).sum(), ok.size), flush=True)
    if ok.any():
        assert_close(got[ok], ref[ok], mag[ok], "f32", l2, what)


# tiles of 16 (whole rows of four channels, and not), of 32 in each shape, the last round cut into parts, the parity classes of stride
# 2; weight gradients of one and two tiles per side, of the first layer's (tap, channel) columns, of one split
@pytest.mark.parametrize("shape", [
    (8, 32, 32, 16, 16, 1), (2, 11, 13, 48, 24, 1), (2, 9, 9, 33, 65, 1), (8, 80, 78, 33, 32, 1), (5, 72, 46, 17, 128, 1), (12, 28, 28, 64, 128, 1),
    (3, 7, 7, 40, 130, 2), (9, 56, 57, 24, 100, 2), (5, 9, 2, 4, 97, 1), (2, 31, 29, 3, 48, 1), (4, 13, 13, 1, 70, 2), (1, 1, 1, 8, 32, 2),
    (1, 3, 3, 700, 260, 1)])
def test_three_passes(B, ctx, oracle, shape):
    N, H, W, C, F, stride = shape
    case = Case(I.Layer(N, H, W, C, F, stride), "f32", 8, I.kept_per_filter(0.3, C), tag=("nonfinite", shape))
    rng = np.random.default_rng(sum(shape))
    pid, kp, M, Wm = oracle_masks(oracle, case)
    x, dy = spoiled(case.x, rng), spoiled(case.dy, rng)
    ax, ady, aW = np.abs(case.x), np.abs(case.dy), np.abs(Wm)
    print("non-finite", shape, flush=True)
    g = GpuLayer(B, ctx, case)
    try:
        finite_x, finite_dy = g.x, g.dy
        g.x, g.dy = to_dev(x), to_dev(dy)
        y_ref, y_mag = oracle.conv_fwd(x, Wm, stride), oracle.conv_fwd(ax, aW, stride)
        dx_ref, dx_mag = oracle.conv_bwd_data(dy, Wm, x.shape, stride), oracle.conv_bwd_data(ady, aW, x.shape, stride)
        assert not np.isfinite(y_ref).all() and not np.isfinite(dx_ref).all()
        check(g.fwd(), y_ref, y_mag, TOL_L2["f32"], "fwd")
        check(g.bwd_data(), dx_ref, dx_mag, TOL_L2["f32"], "bwd_data")
        # the fused ReLU steps: a NaN is not positive
        import torch
        a, dz = torch.full(y_ref.shape, 7.0, device="cuda"), torch.full(dx_ref.shape, 7.0, device="cuda")
        B.pc_conv_fwd_relu(ctx, g.desc, g.pk, g.x, a)
        B.pc_conv_bwd_data_relu(ctx, g.desc, g.pk, g.dy, finite_x, dz)
        torch.cuda.synchronize()
        y, dx = g.fwd(), g.bwd_data()
        assert np.array_equal(a.cpu().numpy(), np.where(y > 0, y, np.float32(0)))
        assert np.array_equal(dz.cpu().numpy(), np.where(case.x > 0, dx, np.float32(0)), equal_nan=True)
        # weight gradients with one side spoiled at a time
        sf, sc = oracle.compact_order(pid, kp, case.P)
        mag = oracle.gather_compact(oracle.conv_bwd_weight(ax, ady, M, stride), pid, case.lib, sf, sc)
        for xs, ds in ((x, case.dy), (case.x, dy)):
            g.x, g.dy = (to_dev(x), finite_dy) if xs is x else (finite_x, to_dev(dy))
            ref = oracle.gather_compact(oracle.conv_bwd_weight(xs, ds, M, stride), pid, case.lib, sf, sc)
            check(g.bwd_weight()[0], ref, mag, TOL_L2_DW, "bwd_weight")
        # a kept weight that is infinite, and one that is pruned away
        W2 = case.W.copy()
        kept, gone = np.argwhere(M != 0), np.argwhere(M == 0)
        W2[tuple(kept[len(kept) // 2])], W2[tuple(gone[len(gone) // 3])] = np.inf, np.nan
        Wm2 = np.where(M != 0, W2, np.float32(0))
        B.pc_update_values(ctx, g.pk, to_dev(W2))
        g.x, g.dy = finite_x, finite_dy
        check(g.fwd(), oracle.conv_fwd(case.x, Wm2, stride), y_mag, TOL_L2["f32"], "fwd, infinite weight")
        check(g.bwd_data(), oracle.conv_bwd_data(case.dy, Wm2, x.shape, stride), dx_mag, TOL_L2["f32"], "bwd_data, infinite weight")
    finally:
        g.close()


@pytest.mark.parametrize("shape", [(8, 80, 78, 33, 32, 1), (12, 28, 28, 64, 128, 1), (9, 56, 57, 24, 100, 2)])
def test_values_that_round_up_to_a_bfloat16_infinity(B, ctx, oracle, shape):
    """3.4e38 is finite in float32 and its leading part of 8 bits is not: the sums that hold such an element are float32's all the same."""
    N, H, W, C, F, stride = shape
    case = Case(I.Layer(N, H, W, C, F, stride), "f32", 8, I.kept_per_filter(0.3, C), tag=("huge", shape))
    rng = np.random.default_rng(sum(shape))
    pid, kp, M, Wm = oracle_masks(oracle, case)
    x, dy = case.x.copy(), (case.dy * np.float32(2.0 ** -10)).astype(np.float32)
    flat = x.reshape(-1, C)
    for p in [0, len(flat) - 1] + list(rng.integers(0, len(flat), size=4)):
        flat[p, rng.integers(0, C)] = np.float32(3.4e38)
    small = np.float32(2.0 ** -10)
    g = GpuLayer(B, ctx, case)
    try:
        g.x, g.dy = to_dev(x), to_dev(dy)
        B.pc_update_values(ctx, g.pk, to_dev((case.W * small).astype(np.float32)))
        y_ref = oracle.conv_fwd(x, (Wm * small).astype(np.float32), stride)
        y_mag = oracle.conv_fwd(np.abs(x), np.abs(Wm * small).astype(np.float32), stride)
        assert np.isfinite(y_ref).all()
        check(g.fwd(), y_ref, y_mag, TOL_L2["f32"], "fwd, huge")
        sf, sc = oracle.compact_order(pid, kp, case.P)
        ref = oracle.gather_compact(oracle.conv_bwd_weight(x, dy, M, stride), pid, case.lib, sf, sc)
        mag = oracle.gather_compact(oracle.conv_bwd_weight(np.abs(x), np.abs(dy), M, stride), pid, case.lib, sf, sc)
        assert np.isfinite(ref).all()
        check(g.bwd_weight()[0], ref, mag, TOL_L2_DW, "bwd_weight, huge")
    finally:
        g.close()
