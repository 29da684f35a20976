"""Stored outputs that lie in the call's own X or W: calls of few tiles, d_in in shares, whose store comes behind every read.  Up to and past 64
128 x 128 tiles, a d_in that its slices do not fill; the bits of a call whose tensors are apart."""
import pytest
import torch

from launches import kernels
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


@pytest.mark.parametrize("over", ["x", "x_columns", "x_row", "w"])
@pytest.mark.parametrize("n,d,r", [(256, 1024, 4), (385, 2048, 16), (1030, 1032, 1), (200, 2056, 17)])
def test_output_over_an_operand(n, d, r, over):
    g, stream = _gen(n), torch.cuda.Stream()
    ctx = binding.Context(stream)
    x, w = (torch.randn(t, d, device="cuda", generator=g).bfloat16() for t in (n, d))
    b = torch.linalg.qr(torch.randn(d, r, device="cuda", generator=g))[0].contiguous()
    apart = torch.empty(n, d, device="cuda", dtype=torch.bfloat16)

    def call(X, W, Y, eps):
        L = binding.make_layer(W, X, r, Y=Y)
        if eps == 0.0:
            ctx.layer_forward_sketch(L, W, X, Y, binding.SKETCH_NONE, None, 0, None, None, None)
        else:
            ctx.perturbed_forward(L, W, X, b, 5, eps, Y, None, None)

    def placed():
        """x, w and the output in their places"""
        buf = torch.zeros((max(n, d) + 1) * (d + 8), device="cuda", dtype=torch.bfloat16)
        held = torch.as_strided(buf, (d if over == "w" else n, d), (d + 8, 1)).copy_(w if over == "w" else x)
        at = {"x": 0, "x_columns": 8, "x_row": d + 8, "w": 0}[over]
        out = torch.as_strided(buf, (n, d), (d + 8, 1), at)
        return (x, held, out) if over == "w" else (held, w, out)
    for eps in (0.0, 1e-2):
        torch.cuda.synchronize()
        call(x, w, apart, eps)
        X, W, out = placed()
        torch.cuda.synchronize()
        call(X, W, out, eps)
        ctx.check()
        assert torch.equal(out, apart), eps
        names, _ = kernels(stream, lambda: call(X, W, out, eps))
        assert sum("gemm_bf16_mid_finish" in s for s in names) == 1 and not any("gemm_bf16_few" in s for s in names), names
        names, _ = kernels(stream, lambda: call(x, w, apart, eps))
        assert sum("gemm_bf16_few_kernel" in s for s in names) == 1, names


@pytest.mark.parametrize("n,d,r", [(300, 1032, 16), (1100, 1160, 3)])
def test_sketched_output_over_its_input(n, d, r):
    """shares of the 128 x 128 kernel, which also sketches them: the output's bits, and the sketch that the 64 x 64 tiles make up to fp32 sums"""
    g, stream = _gen(n), torch.cuda.Stream()
    ctx = binding.Context(stream)
    x, w = (torch.randn(t, d, device="cuda", generator=g).bfloat16() for t in (n, d))
    apart, over = torch.empty_like(x), x.clone()
    s = [torch.empty(d, r, device="cuda") for _ in range(2)]

    def call(X, Y, S):
        ctx.layer_forward_sketch(binding.make_layer(w, X, r, Y=Y), w, X, Y, binding.SKETCH_RANGE_FUSED, None, 91, S, None, None)
    torch.cuda.synchronize()
    call(x, apart, s[0])
    call(over, over, s[1])
    ctx.check()
    assert torch.equal(over, apart)
    assert (s[0].double() - s[1].double()).norm() < 4e-6 * s[0].double().norm()
    names, _ = kernels(stream, lambda: call(over, over, s[1]))
    assert sum("gemm_bf16_mid_finish" in k for k in names) == 1 and not any("gemm_bf16_few" in k for k in names), names


def test_output_beside_its_input_is_apart():
    """columns of one buffer that X does not have: no shares"""
    buf, w, stream = torch.randn(300, 1024, device="cuda", generator=_gen(1)).bfloat16(), torch.randn(400, 512, device="cuda", generator=_gen(2)).bfloat16(), torch.cuda.Stream()
    ctx, x, y = binding.Context(stream), buf[:, :512], buf[:, 600:1000]
    L = binding.make_layer(w, x, 1, Y=y)

    def call():
        ctx.layer_forward_sketch(L, w, x, y, binding.SKETCH_NONE, None, 0, None, None, None)
    torch.cuda.synchronize()
    call()
    ctx.check()
    names, _ = kernels(stream, call)
    assert sum("gemm_bf16_few_kernel" in s for s in names) == 1, names
