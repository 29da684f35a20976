"""A lone layer whose base forward runs beside its extraction: the bits of a step in one stream (timing a kernel class keeps it there), with
inputs written right before and overwritten right after, and of a replayed capture; a layer that is done sooner without stays in one."""
import pytest
import torch

from paper_2601_17261_amd import binding
from test_gpu_beside import _forks

pytestmark = pytest.mark.gpu
EPS, LR = 1e-3, 1e-2


def _layer(kind, n, d_in, d_out):
    g = torch.Generator(device="cuda").manual_seed(n + d_out)
    x = torch.randn(n, d_in, device="cuda", generator=g).bfloat16()
    w = (torch.randn(d_out, d_in, device="cuda", generator=g) * 0.02).bfloat16()
    if kind == "ce":
        t = torch.randint(-1, d_out, (n,), device="cuda", generator=g, dtype=torch.int32)
        return x, w, t, binding.make_loss(t, kind=binding.LOSS_CE)
    t = torch.randn(n, d_out, device="cuda", generator=g)
    t = t if kind == "f32" else t.bfloat16()
    return x, w, t, binding.make_loss(t)


@pytest.mark.parametrize("kind,n,d_in,d_out,r,flags", [("ce", 700, 1024, 9001, 16, 0), ("ce", 2049, 1032, 8192, 1, binding.ONE_SIDED), ("ce", 512, 2048, 16000, 40, 0),
                                                       ("bf16", 3001, 2048, 4096, 4, 0), ("f32", 3072, 2048, 4096, 16, binding.ONE_SIDED)])
def test_same_bits_as_in_one_stream(kind, n, d_in, d_out, r, flags):
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream)
    x, w, t, loss = _layer(kind, n, d_in, d_out)
    out = torch.zeros(4, dtype=torch.float64, device="cuda")
    layer = binding.make_layer(w, x, r)
    given = [a.clone() for a in (x, w, t)]

    def step():
        ctx.step(layer, w, x, loss, 2, EPS, LR, 11, flags, out)

    def run():          # inputs written on the stream right before, overwritten right after
        with torch.cuda.stream(stream):
            for a, s in zip((x, w, t), given):
                a.copy_(s)
            step()
            got = (out.clone(), w.clone())
            for a in (x, w):
                a.fill_(float("nan"))
            t.fill_(0)
        stream.synchronize()
        return got
    torch.cuda.synchronize()
    run()
    ctx.profile_enable(1 << binding.PROF_FILL)
    want = run()
    ctx.profile_enable(False)
    assert torch.isfinite(want[0]).all()
    for _ in range(3):
        assert all(torch.equal(a, b) for a, b in zip(run(), want))
    assert _forks(stream, step)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        step()
    for _ in range(3):
        for a, s in zip((x, w, t), given):
            a.copy_(s)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[0]) and torch.equal(w, want[1])
        assert torch.isfinite(torch.empty(1 << 20, device="cuda").normal_().sum()).item()
    ctx.check()


@pytest.mark.parametrize("kind,n,d_in,d_out", [("bf16", 432, 1024, 1024), ("bf16", 2048, 2048, 2048), ("ce", 200, 2048, 32000)])
def test_one_stream(kind, n, d_in, d_out):
    """128 x 128 tiles, as many 256 x 256 ones as compute units are idle, fewer tokens than a tile"""
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream)
    x, w, t, loss = _layer(kind, n, d_in, d_out)
    out, layer = torch.zeros(4, dtype=torch.float64, device="cuda"), binding.make_layer(w, x, 1)
    torch.cuda.synchronize()
    ctx.step(layer, w, x, loss, 1, EPS, LR, 11, 0, out)
    ctx.check()
    assert not _forks(stream, lambda: ctx.step(layer, w, x, loss, 1, EPS, LR, 11, 0, out))
