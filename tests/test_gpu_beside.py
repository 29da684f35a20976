"""Sets of layers large enough for their base forwards to run on the context's second stream: to the caller all of it is work on the
context's stream (inputs written there just before, weights and inputs overwritten just after), the results are those of a call per
layer, bit for bit, and a captured step replays."""
import ctypes

import pytest
import torch

from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = 1e-3, 1e-3
# d_in, d_out of five layers: 24 GFLOP a forward on 900 tokens (no tile divides them), squared errors in both tilings
SHAPES = [(1024, 2048), (1536, 1024), (1024, 1024), (512, 3072), (2048, 2560)]


def _inputs(n, seed):
    X = [synth.device_powerlaw_x(seed + i, n, d_in) for i, (d_in, _) in enumerate(SHAPES)]
    return [(x,) + synth.device_weights_and_target(seed + 50 + i, x, d_out) for i, (x, (_, d_out)) in enumerate(zip(X, SHAPES))]


def _items(layers, out, r):
    return [(binding.make_layer(w, x, r), w, x, binding.make_loss(t), 30 + i, out[i], None) for i, (x, w, t) in enumerate(layers)]


@pytest.mark.parametrize("flags", [0, binding.ONE_SIDED])
@pytest.mark.parametrize("n,r", [(900, 1), (900, 8), (2600, 40)])
def test_same_as_a_call_per_layer(n, r, flags):
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream=stream)
    given = _inputs(n, 3)
    assert sum(2 * n * i * o for i, o in SHAPES) > 20e9
    want, out1 = [], torch.zeros(len(given), 4, dtype=torch.float64, device="cuda")
    out = torch.zeros_like(out1)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for i, (x, w, t) in enumerate(given):
            w = w.clone()
            ctx.step(binding.make_layer(w, x, r), w, x, binding.make_loss(t), 3, EPS, LR, 30 + i, flags, out1[i])
            want.append(w)
        layers = [tuple(torch.full_like(a, float("nan")) for a in one) for one in given]
        for k in range(3):
            for one, src in zip(layers, given):          # written on the stream, right before
                for a, s in zip(one, src):
                    a.copy_(s)
            ctx.step_many(_items(layers, out, r), 3, EPS, LR, flags)
            got = [w.clone() for _, w, _ in layers]
            for one in layers:                           # and overwritten right after
                for a in one:
                    a.fill_(float("nan"))
            stream.synchronize()
            assert torch.equal(out, out1), k
            assert all(torch.equal(a, b) for a, b in zip(got, want)), k
    ctx.check()
    ctx.close()


def test_captured():
    r, stream = 8, torch.cuda.Stream()
    ctx = binding.Context(stream=stream)
    layers = _inputs(900, 9)
    w0 = [w.clone() for _, w, _ in layers]
    out = torch.zeros(len(layers), 4, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    ref = []
    with torch.cuda.stream(stream):
        for _ in range(3):
            ctx.step_many(_items(layers, out, r), 3, EPS, LR, 0)
            stream.synchronize()
            ref.append(([w.clone() for _, w, _ in layers], out.clone()))
        for (_, w, _), s in zip(layers, w0):
            w.copy_(s)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            ctx.step_many(_items(layers, out, r), 3, EPS, LR, 0)
    torch.cuda.synchronize()
    assert all(torch.equal(w, s) for (_, w, _), s in zip(layers, w0))
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref[k][1]), k
        assert all(torch.equal(w, s) for (_, w, _), s in zip(layers, ref[k][0])), k
        scratch = torch.empty(1 << 20, device="cuda").normal_()
        assert torch.isfinite(scratch.sum()).item()
    with torch.cuda.stream(stream):
        ctx.step_many(_items(layers, out, r), 3, EPS, LR, 0)      # the context's own streams are as before
        ctx.check()
    ctx.close()


def _forks(stream, call):
    """whether the launches of a call are no single chain: a captured chain has one edge less than nodes"""
    graph, before = torch.cuda.CUDAGraph(keep_graph=True), torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        before.add_(1)          # what the fork follows
        call()
    lib, raw = binding.load(), ctypes.c_void_p(graph.raw_cuda_graph())
    nodes, edges = ctypes.c_size_t(0), ctypes.c_size_t(0)
    assert lib.hipGraphGetNodes(raw, None, ctypes.byref(nodes)) == 0
    assert lib.hipGraphGetEdges(raw, None, None, ctypes.byref(edges)) == 0
    assert nodes.value > 10 and edges.value >= nodes.value - 1
    return edges.value >= nodes.value


def _mixed(n_bf16, n_f32, n_ce, tokens=900, r=4):
    """(W, X, loss with its target) of squared-error layers in bf16, each of 24 GFLOP a forward on 900 tokens, in fp32, and of heads"""
    got = []
    for i in range(n_bf16):
        x = synth.device_powerlaw_x(i, tokens, 2600)
        w, t = synth.device_weights_and_target(50 + i, x, 5200)
        got.append((w, x, t, binding.make_loss(t)))
    for i in range(n_f32):
        w, x, t = (torch.randn(s, device="cuda") for s in ((96, 200), (333, 200), (333, 96)))
        got.append((w, x, t, binding.make_loss(t)))
    for i in range(n_ce):
        w, x = (torch.randn(s, device="cuda").bfloat16() for s in ((1000, 264), (300, 264)))
        t = torch.randint(0, 1000, (300,), device="cuda", dtype=torch.int32)
        got.append((w, x, t, binding.make_loss(t, kind=binding.LOSS_CE)))
    out = torch.zeros(len(got), 4, dtype=torch.float64, device="cuda")
    return got, out, [(binding.make_layer(w, x, r), w, x, loss, 30 + i, out[i], None) for i, (w, x, _, loss) in enumerate(got)]


@pytest.mark.parametrize("n_bf16,n_f32,n_ce,forks", [(4, 0, 0, True), (1, 3, 0, False), (1, 0, 3, False), (2, 2, 2, False), (3, 1, 0, False), (4, 1, 1, True)])
def test_the_layers_that_count(n_bf16, n_f32, n_ce, forks):
    """two streams pay from four layers on whose forwards run on the second one; other layers of the list are not among them"""
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream=stream)
    _, _, items = _mixed(n_bf16, n_f32, n_ce)
    torch.cuda.synchronize()

    def call():
        ctx.step_many(items, 3, EPS, LR, 0)
    with torch.cuda.stream(stream):
        call()
        stream.synchronize()
    assert _forks(stream, call) == forks
    ctx.check()
    ctx.close()


# four layers of 77 GFLOP a forward, in 128 x 128 tiles: longer than one column's extraction, not than 64 columns'; in the other tiling
# nothing is left waiting on half of the compute units
@pytest.mark.parametrize("r,K,large,forks", [(1, 3, False, False), (1, 6, False, True), (64, 3, False, True), (64, 0, False, False), (1, 3, True, True)])
def test_forwards_that_outlast_the_extraction(r, K, large, forks):
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream=stream)
    x = torch.randn(768, 4096, device="cuda").bfloat16()
    w, t = torch.randn(12288, 4096, device="cuda").bfloat16(), torch.randn(768, 12288, device="cuda").bfloat16()
    layer = binding.make_layer(w, x, r)
    layer.tiling = binding.TILING_LARGE if large else binding.TILING_AUTO
    out = torch.zeros(4, 4, dtype=torch.float64, device="cuda")
    b = torch.empty(4, 4096, r, device="cuda")
    items = [(layer, w, x, binding.make_loss(t), i, out[i], b[i]) for i in range(4)]
    torch.cuda.synchronize()

    def call():
        ctx.step_many(items, K, EPS, LR, 0)
    with torch.cuda.stream(stream):
        call()
        stream.synchronize()
    assert _forks(stream, call) == forks
    ctx.check()
    ctx.close()


@pytest.mark.parametrize("n_bf16,n_f32,n_ce,tokens,r", [(4, 1, 1, 900, 4), (5, 2, 3, 900, 1), (18, 1, 1, 400, 8), (17, 0, 0, 400, 40)])
def test_beside_layers_of_other_kinds(n_bf16, n_f32, n_ce, tokens, r):
    """base forwards on the second stream while those of fp32 layers and heads, and the extraction of all, run on the context's; also more
    of them than a launch takes.  Written right before, overwritten right after: the bits of a call per layer"""
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream=stream)
    layers, out, items = _mixed(n_bf16, n_f32, n_ce, tokens, r)
    given = [(w.clone(), x.clone(), t.clone()) for w, x, t, _ in layers]
    want, out1 = [], torch.zeros_like(out)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for i, ((w, x, t), (_, _, _, loss)) in enumerate(zip(given, layers)):
            w = w.clone()
            own = binding.make_loss(t, kind=loss.kind)
            ctx.step(binding.make_layer(w, x, r), w, x, own, 3, EPS, LR, 30 + i, 0, out1[i])
            want.append(w)
        ctx.step_many(items, 3, EPS, LR, 0)
        for _ in range(3):
            for (w, x, t, _), src in zip(layers, given):
                for a, s in zip((w, x, t), src):
                    a.copy_(s)
            out.fill_(float("nan"))
            ctx.step_many(items, 3, EPS, LR, 0)
            got = [w.clone() for w, _, _, _ in layers]
            for w, x, t, _ in layers:
                w.fill_(float("nan"))
                x.fill_(float("nan"))
                t.fill_(-1 if t.dtype == torch.int32 else float("nan"))
            stream.synchronize()
            assert torch.equal(out, out1)
            assert all(torch.equal(a, b) for a, b in zip(got, want))
    ctx.check()
    assert _forks(stream, lambda: ctx.step_many(items, 3, EPS, LR, 0))
    ctx.close()
