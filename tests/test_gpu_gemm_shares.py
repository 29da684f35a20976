"""Stored outputs of few 128 x 128 tiles and a d_in too deep for 64 x 64 ones, which is walked in shares: two (96 tiles), four, five and eight of
them, slices that the shares do not divide, a last slice that d_in does not fill, a rank-r term behind the last share, shifted last tiles.
Tolerances as in test_gpu_gemm_mid.py."""
import numpy as np
import pytest
import torch

from launches import kernels
from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS = float(np.float32(1e-2))


@pytest.mark.parametrize("n,d_out,d_in,r", [(128, 128, 2560, 1), (385, 2048, 2632, 16), (129, 300, 4168, 17), (500, 131, 2200, 64), (1000, 1500, 3096, 4)])
def test_stored_output(n, d_out, d_in, r):
    W, X, _ = synth.single_layer_problem(5, n, d_in, d_out, kind="rmsnorm", storage="bf16")
    Wd, Xd = torch.from_numpy(W).cuda().to(torch.bfloat16), torch.from_numpy(X).cuda().to(torch.bfloat16)
    B = torch.linalg.qr(torch.randn(d_in, r, device="cuda", generator=torch.Generator(device="cuda").manual_seed(r)))[0].contiguous()
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream)
    Y0 = X.astype(np.float64) @ W.astype(np.float64).T
    D = (X.astype(np.float64) @ B.double().cpu().numpy()) @ oagzo.gaussian_factor(5, d_out, r).T
    for eps in (0.0, EPS, -EPS):
        Y = torch.full((n, d_out), 7.0, device="cuda", dtype=torch.bfloat16)
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
        names, _ = kernels(stream, call)
        assert sum("gemm_bf16_mid_kernel" in s for s in names) == 1 and sum("gemm_bf16_mid_finish" in s for s in names) == 1, names
