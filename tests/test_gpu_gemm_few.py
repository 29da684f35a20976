"""Stored outputs of few tiles whose waves share d_in (gemm_bf16_few.hip) at the edges of its range: one slice a wave and shares that differ,
a slice that d_in does not fill, shifted last tiles, one and two workgroups to a compute unit, extension slices behind the last share; and
that the sides of its line go where they should.  Tolerances as in test_gpu_gemm_mid.py."""
import numpy as np
import pytest
import torch

from launches import kernels
from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS = float(np.float32(1e-2))


@pytest.mark.parametrize("n,d_out,d_in,r", [(128, 128, 256, 1), (129, 131, 264, 16), (191, 200, 328, 17), (1024, 1024, 320, 4), (1025, 1030, 712, 64),
                                            (130, 2000, 2048, 33), (260, 1100, 2552, 8), (1025, 1030, 824, 4), (1025, 1030, 1032, 1), (1025, 1030, 2040, 16),
                                            (598, 3238, 1352, 2)])
def test_stored_output(n, d_out, d_in, r):
    W, X, _ = synth.single_layer_problem(5, n, d_in, d_out, kind="rmsnorm", storage="bf16")

    def strided(a, pad):
        t = torch.full((a.shape[0], a.shape[1] + pad), float("nan"), device="cuda", dtype=torch.bfloat16)[:, :a.shape[1]]
        return t.copy_(torch.from_numpy(a))
    Wd, Xd = strided(W, 16), strided(X, 8)
    B = torch.linalg.qr(torch.randn(d_in, r, device="cuda", generator=torch.Generator(device="cuda").manual_seed(r)))[0].contiguous()
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream)
    torch.cuda.synchronize()
    Y0 = X.astype(np.float64) @ W.astype(np.float64).T
    D = (X.astype(np.float64) @ B.double().cpu().numpy()) @ oagzo.gaussian_factor(5, d_out, r).T
    for eps in (0.0, EPS, -EPS):
        buf = torch.full((n, d_out + 3), 7.0, device="cuda", dtype=torch.bfloat16)
        Y = buf[:, :d_out]
        L = binding.make_layer(Wd, Xd, r, Y=Y)

        def call():
            if eps == 0.0:
                ctx.layer_forward_sketch(L, Wd, Xd, Y, binding.SKETCH_NONE, None, 0, None, None, None)
            else:
                ctx.perturbed_forward(L, Wd, Xd, B, 5, eps, Y, None, None)
        torch.cuda.synchronize()
        call()
        ctx.check()
        want = Y0 + eps * D
        err = np.abs(Y.double().cpu().numpy() - want)
        assert np.all(err <= 2.0 ** -8 * np.abs(want) + 1e-5 * np.sqrt(np.mean(want ** 2))), eps
        assert bool((buf[:, d_out:] == 7.0).all())
        names, _ = kernels(stream, call)
        assert sum("gemm_bf16_few_kernel" in s for s in names) == 1 and not any("gemm_bf16_mid" in s for s in names), names


@pytest.mark.parametrize("n,d_out,d_in", [(128, 128, 248), (1088, 1984, 512), (300, 300, 2056), (512, 512, 2568), (1025, 1030, 840), (1025, 1030, 1016),
                                          (1025, 1030, 2056), (598, 3238, 1336)])
def test_beyond_the_line(n, d_out, d_in):
    """d_in of fewer than four slices, 527 tiles, 25 tiles of more than 32 slices, 64 of more than 40, and, of rows that do not start on 128 bytes, more than
    256 tiles of 13 to 15 slices, of more than 32, and of up to 20 where there are more than 128 tiles of 128 x 128: these"""
    g = torch.Generator(device="cuda").manual_seed(d_in)
    x, w = torch.randn(n, d_in, device="cuda", generator=g).bfloat16(), torch.randn(d_out, d_in, device="cuda", generator=g).bfloat16()
    stream = torch.cuda.Stream()
    ctx, y = binding.Context(stream), torch.empty(n, d_out, device="cuda", dtype=torch.bfloat16)
    L = binding.make_layer(w, x, 1, Y=y)

    def call():
        ctx.layer_forward_sketch(L, w, x, y, binding.SKETCH_NONE, None, 0, None, None, None)
    torch.cuda.synchronize()
    call()
    ctx.check()
    want = x.double() @ w.double().T
    assert ((y.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * want.square().mean().sqrt()).all()
    names, _ = kernels(stream, call)
    assert any("gemm_bf16_mid_kernel" in s for s in names) and not any("gemm_bf16_few" in s for s in names), names


# one slice a wave and two tiles that share them out; shifted tiles, one and two workgroups to a compute unit; more tiles than slices, which then sketch
# nothing; partial sums of 128 token tiles; more slices than tiles and a last one that d_in does not fill
@pytest.mark.parametrize("n,d_out,d_in,r", [(128, 128, 256, 16), (191, 200, 328, 7), (1025, 1030, 712, 16), (130, 2000, 2048, 1), (8192, 256, 264, 3), (300, 130, 2040, 13)])
def test_sketched(n, d_out, d_in, r):
    """the output's bits with and without the sketch, and the sketch against fp64: sums of 64 products and of their roundings, as in
    test_gpu_sketch_rings.py, whose sums are longer"""
    W, X, _ = synth.single_layer_problem(5, n, d_in, d_out, kind="rmsnorm", storage="bf16")
    Xd = torch.full((n, d_in + 8), float("nan"), device="cuda", dtype=torch.bfloat16)[:, :d_in].copy_(torch.from_numpy(X))
    Wd = torch.from_numpy(W).cuda().to(torch.bfloat16)
    stream = torch.cuda.Stream()
    ctx, got = binding.Context(stream), []
    for mode in (binding.SKETCH_NONE, binding.SKETCH_RANGE_FUSED):
        Y, S = torch.full((n, d_out), 7.0, device="cuda", dtype=torch.bfloat16), torch.full((d_in, r), 9.0, device="cuda")
        L = binding.make_layer(Wd, Xd, r, Y=Y)

        def call():
            ctx.layer_forward_sketch(L, Wd, Xd, Y, mode, None, 91, S, None, None)
        torch.cuda.synchronize()
        call()
        ctx.check()
        names, _ = kernels(stream, call)
        assert sum("gemm_bf16_few_kernel" in s for s in names) == 1 and not any("gemm_bf16_mid" in s for s in names), names
        got.append(Y)
    assert torch.equal(got[0], got[1])
    want = oagzo.range_sketch(X.astype(np.float64), r, 91)
    assert np.linalg.norm(S.double().cpu().numpy() - want) < 4e-6 * np.linalg.norm(want)
