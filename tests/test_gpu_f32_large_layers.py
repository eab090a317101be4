"""Float32 layers of more than 102400 kernels, whose packs hold no weights in three parts: the kernels in tiles of 32 split them as they go.
Every arrangement of the wavefronts in both passes and at both strides, rows that are no whole quads, last rounds cut into parts, element by
element against the oracle; and the same bits as over weights that are split in the pack."""
import numpy as np
import pytest

from paper_2011_10170_amd import inputs as I
from tests._harness import Case, GpuLayer, assert_close, oracle_masks, TOL_L2

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


# (pass, arrangement, layer); forward: the last round cut into parts in the second of each pair at stride 1
@pytest.mark.parametrize("what,waves,shape", [
    ("fwd", "1, 1, 4, 1", (2, 11, 11, 132, 776, 1)), ("fwd", "1, 1, 4, 1", (4, 14, 14, 512, 512, 1)), ("fwd", "1, 1, 4, 1", (1, 23, 22, 134, 766, 2)),
    ("fwd", "1, 4, 1, 1", (3, 17, 20, 101, 1021, 1)), ("fwd", "1, 4, 1, 1", (1, 42, 40, 160, 643, 1)),
    ("fwd", "1, 4, 1, 2", (4, 38, 37, 145, 712, 1)), ("fwd", "1, 4, 1, 2", (4, 38, 37, 144, 714, 1)),
    ("fwd", "2, 2, 1, 1", (2, 19, 22, 100, 1025, 1)), ("fwd", "2, 2, 1, 1", (2, 22, 24, 110, 931, 1)), ("fwd", "2, 2, 1, 1", (9, 17, 20, 100, 1025, 2)),
    ("fwd", "2, 2, 1, 2", (6, 19, 19, 107, 958, 1)), ("fwd", "2, 2, 1, 2", (2, 33, 33, 108, 949, 1)),
    ("fwd", "4, 1, 1, 1", (2, 28, 28, 320, 328, 1)), ("fwd", "4, 1, 1, 1", (1, 31, 33, 114, 903, 1)), ("fwd", "4, 1, 1, 1", (22, 13, 11, 100, 1026, 2)),
    ("fwd", "4, 1, 1, 2", (1, 54, 54, 100, 1025, 1)), ("fwd", "4, 1, 1, 2", (6, 18, 18, 103, 1002, 1)), ("fwd", "4, 1, 1, 2", (18, 20, 21, 103, 1001, 2)),
    ("bwd", "1, 1, 4, 1", (3, 8, 7, 684, 151, 1)), ("bwd", "1, 4, 1, 1", (3, 18, 18, 916, 112, 1)), ("bwd", "1, 4, 1, 2", (1, 67, 68, 781, 139, 1)),
    ("bwd", "2, 2, 1, 1", (2, 20, 22, 976, 105, 1)), ("bwd", "2, 2, 1, 2", (1, 51, 51, 801, 132, 1)), ("bwd", "4, 1, 1, 1", (13, 6, 7, 996, 104, 1)),
    ("bwd", "4, 1, 1, 2", (1, 44, 45, 904, 118, 1)),
    ("bwd", "1, 4, 1, 1", (6, 14, 16, 668, 155, 2)), ("bwd", "1, 4, 1, 2", (2, 51, 52, 648, 168, 2)), ("bwd", "2, 2, 1, 1", (1, 23, 23, 855, 121, 2)),
    ("bwd", "2, 2, 1, 2", (1, 44, 44, 724, 142, 2)), ("bwd", "4, 1, 1, 1", (2, 11, 12, 920, 120, 2)), ("bwd", "4, 1, 1, 2", (1, 28, 29, 952, 111, 2))])
def test_weights_split_in_the_kernel(B, ctx, oracle, what, waves, shape):
    L = I.Layer(*shape)
    assert L.F * L.C > 102400
    case = Case(L, "f32", 8, I.kept_per_filter(0.3, L.C), tag=("large", what, shape))
    Wm = oracle_masks(oracle, case)[3]
    g = GpuLayer(B, ctx, case)
    try:
        got = g.fwd() if what == "fwd" else g.bwd_data()
        name = B.pc_last_kernel(ctx)
    finally:
        g.close()
    assert name.startswith("pc_f32_conv_kernel<32, %s, " % waves) and name.endswith(", false>"), name
    run = (lambda a, w: oracle.conv_fwd(a, w, L.stride)) if what == "fwd" else (lambda a, w: oracle.conv_bwd_data(a, w, case.x.shape, L.stride))
    src = case.x if what == "fwd" else case.dy
    assert_close(got, run(src, Wm), run(np.abs(src), np.abs(Wm)), "f32", TOL_L2["f32"], what)


@pytest.mark.parametrize("what,shape,more", [
    ("fwd", (3, 32, 32, 224, 448, 1), 458), ("bwd", (3, 32, 32, 224, 448, 1), 458), ("bwd", (3, 32, 32, 224, 448, 2), 458), ("fwd", (1, 54, 54, 100, 1024, 1), 1025),
    ("fwd", (4, 38, 37, 144, 704, 1), 714), ("bwd", (4, 38, 37, 144, 704, 1), 714), ("bwd", (9, 30, 31, 256, 400, 1), 402)])
def test_the_same_bits_as_split_in_the_pack(B, ctx, what, shape, more):
    """A layer of up to 102400 kernels, and the same with a few filters more, whose errors are zero: sums run over the channels in groups of 16,
    the taps of a group in order, whatever the tile (where wavefronts share no reduction), and products with zero add nothing."""
    import torch
    N, H, W, C, F, st = shape
    lib, k = I.make_library(8), I.kept_per_filter(0.4, C)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(F + C + st)
    L = I.Layer(*shape)
    w, x = torch.randn((more, C, 9), generator=gen, device="cuda"), torch.randn((N, H, W, C), generator=gen, device="cuda")
    dy = torch.zeros((N, L.Ho, L.Wo, more), device="cuda")
    dy[..., :F] = torch.randn((N, L.Ho, L.Wo, F), generator=gen, device="cuda")
    pid, keep = (torch.zeros((more, C), dtype=torch.uint8, device="cuda") for _ in range(2))
    B.pc_pattern_select(ctx, w, None, more, C, lib, B.PC_KEEP_PER_FILTER, k, B.PC_SCORE_RETAINED, pid, keep)
    out = []
    for f in (F, more):
        pk = B.pc_pack(ctx, w[:f].contiguous(), pid[:f].contiguous(), keep[:f].contiguous(), f, C, lib, B.PC_F32)
        d = B.make_desc(N, H, W, C, f, st, B.PC_F32)
        if what == "fwd":
            o = torch.full((N, L.Ho, L.Wo, f), float("nan"), device="cuda")
            B.pc_conv_fwd(ctx, d, pk, x, o)
            out.append(o[..., :F])
        else:
            o = torch.full((N, H, W, C), float("nan"), device="cuda")
            B.pc_conv_bwd_data(ctx, d, pk, dy[..., :f].contiguous(), o)
            out.append(o)
        name = B.pc_last_kernel(ctx)
        v = name[len("pc_f32_conv_kernel<"):-1].split(", ")      # tile, wavefronts by channels, pixels, reduction, ...; whether the pack holds the parts
        assert v[0] == "32" and v[3] == "1" and v[-1] == ("true" if f == F else "false"), name
        B.pc_packed_free(pk)
    assert torch.equal(out[0], out[1])
