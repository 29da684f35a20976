"""The projection of a perturbed forward for up to 16 columns, multiplied from the fp32 basis in 64-wide slices that eight waves share:
fewer slices than waves, slices that d_in does not fill, tokens that workgroups do not divide, columns short of 16, an unaligned basis."""
import pytest
import torch

from oracle import agzo as oagzo
from launches import kernels
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,r", [(2, 8, 2), (31, 64, 3), (33, 72, 16), (65, 504, 5), (40, 512, 16), (385, 1032, 2), (129, 2048, 16), (96, 4104, 9), (4700, 4104, 9), (8192, 24, 1),
                                   (8225, 136, 16)])
def test_projection(n, d, r):
    """Y = eps (X B) G^T with W = 0: X B in fp32 sums of d exact products, sqrt(d) 2^-24 of |x| |b| at most; the rank-r term as bf16
    hi / lo pairs (2^-16 of each of its r terms), stored as bf16"""
    ctx = binding.Context()
    X = torch.full((n, d + 8), float("nan"), device="cuda", dtype=torch.bfloat16)[:, :d]      # (nothing behind d_in is read as a value)
    X.copy_(torch.randn(n, d, device="cuda"))
    B = torch.empty(d * r + 1, device="cuda")[1:].view(d, r)
    B.copy_(torch.randn(d, r, device="cuda"))
    W = torch.zeros(140, d, device="cuda", dtype=torch.bfloat16)
    got = []
    for mask in (0, binding.PROF_ALL):
        Y = torch.full((n, 140), 7.0, device="cuda", dtype=torch.bfloat16)
        ctx.profile_enable(mask)
        ctx.perturbed_forward(binding.make_layer(W, X, r, Y=Y), W, X, B, 9, 0.5, Y, None, None)
        ctx.check()
        got.append(Y)
    assert torch.equal(*got)
    G = torch.from_numpy(oagzo.gaussian_factor(9, 140, r)).cuda().double()
    want = 0.5 * (X.double() @ B.double()) @ G.T
    size = 0.5 * (X.double().norm(dim=1, keepdim=True) * B.double().norm(dim=0)) @ G.abs().T
    assert ((got[0].double() - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -15 * size).all()


# one round of workgroups of 32 tokens, d_in in no more shares than eight where it would be split otherwise
@pytest.mark.parametrize("n,d,r,one", [(385, 2048, 16, True), (128, 2056, 16, False), (2313, 2056, 2, True), (2312, 2056, 2, False), (385, 6144, 16, False), (6912, 6144, 4, True),
                                       (8192, 512, 16, True), (8193, 512, 16, False), (8192, 8192, 16, False), (385, 2048, 17, False)])
def test_which_launches(n, d, r, one):
    stream = torch.cuda.Stream()
    ctx = binding.Context(stream=stream)
    X, W = torch.zeros(n, d, device="cuda", dtype=torch.bfloat16), torch.zeros(8, d, device="cuda", dtype=torch.bfloat16)
    B, Y = torch.zeros(d, r, device="cuda"), torch.empty(n, 8, device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()

    def call():
        ctx.perturbed_forward(binding.make_layer(W, X, r, Y=Y), W, X, B, 9, 0.5, Y, None, None)
    with torch.cuda.stream(stream):
        call()
        stream.synchronize()
    names, _ = kernels(stream, call)
    assert any("xq_ext_kernel" in name for name in names) == one, names
    assert any("xq_bf16_many" in name or "xq_direct" in name for name in names) != one, names
    ctx.close()
