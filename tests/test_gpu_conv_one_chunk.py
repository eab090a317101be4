"""The register kernels that split the reduction over their wavefronts, on layers of one channel chunk and several tiles per workgroup: every
item ends a tile, so the area through which the wavefronts add their sums is written again one item after it was read. (A wavefront that
owned no part of the tile could overwrite it before the owners had read it.)"""
import pytest

from paper_2011_10170_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [7, 8, 9, 14, 15, 21, 27, 28, 29])
@pytest.mark.parametrize("dims", [(24, 32, 32, 64, 128), (60, 16, 16, 24, 264)])
def test_same_sums_every_time(cfg, dims):
    import torch
    from paper_2011_10170_amd import binding as B
    from tests._harness import Case, GpuLayer
    B.load()
    ctx = B.pc_create(0, torch.cuda.current_stream().cuda_stream)
    L = I.Layer(*dims, 1)
    g = GpuLayer(B, ctx, Case(L, "bf16", 8, I.kept_per_filter(0.3, L.C), tag=("one_chunk", "x")))
    try:
        y = torch.empty((L.N, L.Ho, L.Wo, L.F), dtype=torch.bfloat16, device="cuda")
        B.pc_set_plan_override(ctx, 20, 0)      # the pixel split: another order of additions, at most a unit in the last place apart
        B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, y)
        want = y.double()
        B.pc_set_plan_override(ctx, cfg, 0)
        first = None
        for _ in range(20):
            y.fill_(float("nan"))
            B.pc_conv_fwd(ctx, g.desc, g.pk, g.x, y)
            if first is None:
                first = y.clone()
                a = y.double()
                assert bool((a - want).abs().le(2.0 ** -7 * torch.maximum(a.abs(), want.abs()) + 2.0 ** -12 * want.abs().max()).all())
            assert torch.equal(y.view(torch.int16), first.view(torch.int16))
    finally:
        B.pc_set_plan_override(ctx, -1, 0)
        g.close()
        B.pc_destroy(ctx)
