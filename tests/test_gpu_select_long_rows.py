"""Selection of rows of 513 .. 8192 kernels (a workgroup per row, keys in LDS): bit-exact against the oracle at the edges of its
range, one launch per 32 layers, and no device memory of its own, so that the first call of a context can be captured."""
import ctypes

import numpy as np
import pytest

from paper_2011_10170_amd import inputs as I
from tests._harness import to_dev

pytestmark = pytest.mark.gpu

LIB = I.make_library(12)


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2011_10170_amd import binding
    binding.load()
    return binding


def layers(oracle, shapes, ties):
    """Per layer: weights, gradients (every third layer has none), kept kernels, and the oracle's selection."""
    out = []
    for l, (F, C) in enumerate(shapes):
        if ties:
            rng = np.random.default_rng(F * 7 + C + l)
            W, G = (rng.integers(-2, 3, size=(F, C, 9)).astype(np.float32) * 0.5 for _ in range(2))
        else:
            W, G = I.gen_weights(F, C, I.BASE_SEED, ("long", l)), I.gen_weight_grads(F, C, I.BASE_SEED, ("long", l))
        G = None if l % 3 == 2 else G
        n_keep = (C // 3, 1, C - 1, C, 0)[l % 5]
        out.append((W, G, n_keep) + oracle.select(W, G, LIB, n_keep, keep_mode=0, score_mode=0))
    return out


def select(B, ctx, want):
    """The batch call on device copies of the layers; (call, pid, keep)."""
    import torch
    W, G = [to_dev(w[0]) for w in want], [None if w[1] is None else to_dev(w[1]) for w in want]
    F, C = [w.shape[0] for w in W], [w.shape[1] for w in W]
    pid, keep = ([torch.full((f, c), 255, dtype=torch.uint8, device="cuda") for f, c in zip(F, C)] for _ in range(2))
    return lambda: B.pc_pattern_select_batch(ctx, W, G, F, C, LIB, 0, [w[2] for w in want], 0, pid, keep), pid, keep


def check(want, pid, keep):
    for l, w in enumerate(want):
        assert np.array_equal(pid[l].cpu().numpy(), w[3]), l
        assert np.array_equal(keep[l].cpu().numpy(), w[4]), l


@pytest.mark.parametrize("ties", [False, True])
def test_edges_of_the_range(B, oracle, ties):
    import torch
    # one chunk past the registers' range, whole and cut chunks of 64 and of 512, both ends of the range and the first row past it
    # (scores in memory), short rows among them
    want = layers(oracle, [(5, 513), (3, 576), (2, 700), (70, 512), (4, 1024), (3, 1025), (2, 4097), (9, 65), (3, 8191), (2, 8192), (1, 8193)], ties)
    ctx = B.pc_create(0, torch.cuda.current_stream().cuda_stream)
    try:
        run, pid, keep = select(B, ctx, want)
        run()
        torch.cuda.synchronize()
        check(want, pid, keep)
    finally:
        B.pc_destroy(ctx)


@pytest.mark.parametrize("shape", [(300, 1024), (2, 1025), (256, 1100), (257, 1100), (1, 8192)])
def test_one_layer_of_few_or_many_rows(B, oracle, shape):
    import torch
    want = layers(oracle, [shape], True)
    ctx = B.pc_create(0, torch.cuda.current_stream().cuda_stream)
    try:
        run, pid, keep = select(B, ctx, want)
        run()
        torch.cuda.synchronize()
        check(want, pid, keep)
    finally:
        B.pc_destroy(ctx)


def graph_nodes(graph):
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    n = ctypes.c_size_t()
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# 40 layers: 32 and 8; one layer of few long rows, whose scores go through memory where that needs no allocation
@pytest.mark.parametrize("shapes, launches", [([(2 + l % 3, 520 + 97 * l) for l in range(40)], 2), ([(5, 3001)], 1)])
def test_one_launch_per_32_layers_and_no_scratch(B, oracle, shapes, launches):
    import torch
    want = layers(oracle, shapes, False)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = B.pc_create(0, stream.cuda_stream)
        run, pid, keep = select(B, ctx, want)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g, stream=stream):
            run()                               # the context's first call: an allocation here fails the capture
        assert graph_nodes(g) == launches
        g.instantiate()
        for _ in range(3):
            for t in pid + keep:
                t.fill_(255)
            g.replay()
            torch.cuda.synchronize()
            check(want, pid, keep)
    B.pc_destroy(ctx)
