"""X Q for a single column on the vector units: widths below, at and past the chunks that waves share, tokens that waves and workgroups
do not divide, unaligned factors, every output form."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu

SHAPES = [(1, 8), (3, 64), (17, 504), (33, 512), (66, 520), (5, 1024), (129, 1032), (7, 1536), (9, 1544), (40, 2560), (21, 4104), (8191, 16), (8192, 16)]


def _offset(a, k):
    """the same values k floats behind a 16-byte boundary"""
    flat = torch.empty(a.numel() + 4, device="cuda")
    v = flat[k:k + a.numel()].view(a.shape)
    v.copy_(a)
    return v


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n,d", SHAPES)
def test_sketch_and_perturbed_forward(n, d, shift):
    """T = X q in fp32 sums of at most d terms: sqrt(d) 2^-24 of |x| |q|; the sketch adds n of them"""
    ctx = binding.Context()
    X = torch.randn(n, d + 8, device="cuda").bfloat16()[:, :d]
    q = _offset(torch.randn(d, 1, device="cuda"), shift)
    S = torch.empty(d, 1, device="cuda")
    ctx.layer_forward_sketch(binding.make_layer(torch.empty(16, d, device="cuda", dtype=torch.bfloat16), X, 1), None, X, None, binding.SKETCH_POWER, q, 0, S, None, None)
    T = X.double() @ q.double()
    want = X.double().T @ T
    tol = 4 * 2.0 ** -24 * ((d ** 0.5) * X.double().abs().T @ (X.double().norm(dim=1, keepdim=True) * q.double().norm() / d ** 0.5) + n ** 0.5 * (X.double().abs().T @ T.abs()))
    assert ((S.double() - want).abs() <= tol + 1e-30).all()
    # the projection inside a forward: Y = eps (X q) G^T with W = 0, rank-r term as bf16 hi / lo pairs (2^-16 of it), stored as bf16
    W = torch.zeros(140, d, device="cuda", dtype=torch.bfloat16)
    Y = torch.full((n, 140), 7.0, device="cuda", dtype=torch.bfloat16)
    ctx.perturbed_forward(binding.make_layer(W, X, 1, Y=Y), W, X, q, 9, 0.5, Y, None, None)
    ctx.check()
    G = torch.from_numpy(oagzo.gaussian_factor(9, 140, 1)).cuda().double()
    want = 0.5 * T @ G.T
    err = (Y.double() - want).abs()
    assert (err <= (2.0 ** -8 + 2.0 ** -14) * want.abs() + 2e-6 * X.double().norm(dim=1, keepdim=True) * q.double().norm() * G.abs().max()).all()


def test_many_layers_as_one_by_one():
    ctx = binding.Context()
    X = [torch.randn(n, d, device="cuda").bfloat16() for n, d in SHAPES]
    lay = [binding.make_layer(torch.empty(16, x.shape[1], device="cuda", dtype=torch.bfloat16), x, 1) for x in X]
    many = [torch.empty(x.shape[1], 1, device="cuda") for x in X]
    ctx.basis_many([(l, x, 3 + i, None, b) for i, (l, x, b) in enumerate(zip(lay, X, many))], 2, 0)
    for i, (l, x, b) in enumerate(zip(lay, X, many)):
        one = torch.empty_like(b)
        ctx.basis(l, x, 2, 3 + i, None, 0, one)
        assert torch.equal(one, b), i
    ctx.check()


@pytest.mark.parametrize("scale", [1.0, 1e-12, 1e12])
@pytest.mark.parametrize("n,d,K", [(300, 1032, 1), (300, 1032, 3), (65, 8, 2), (8191, 264, 2)])
def test_normalised_by_the_projection(n, d, K, scale):
    """Between power steps the column stays as the sketch left it and the projection normalises its result.  From a given first sketch
    of any size, against fp64: each step rounds the column and T to fp32"""
    ctx = binding.Context()
    X = torch.randn(n, d, device="cuda").bfloat16()
    S0 = scale * torch.randn(d, 1, device="cuda")
    B = torch.empty(d, 1, device="cuda")
    ctx.basis(binding.make_layer(torch.empty(16, d, device="cuda", dtype=torch.bfloat16), X, 1), X, K, 3, S0, 0, B)
    ctx.check()
    q = S0.double() / S0.double().norm()
    for _ in range(K):
        q = X.double().T @ (X.double() @ q)
        q = q / q.norm()
    assert (B.double() - q).norm() <= (K + 1) * 4e-6


@pytest.mark.parametrize("of_x,of_s0", [(1e-16, 1.0), (1e-12, 1.0), (1e12, 1.0), (1e16, 1.0), (1.0, 1e-37), (1.0, 1e37), (1e16, 1e37), (1e-16, 1e-37)])
@pytest.mark.parametrize("n,d,K", [(300, 1032, 1), (65, 8, 3), (8191, 264, 2)])
def test_range_of_a_column_left_to_be_normalised(n, d, K, of_x, of_s0):
    """A sketch is of size |X|^2, and so is the column between power steps: activations and first sketches whose squares fp32 holds
    lose nothing, though the product of such a column with X is of size |X|^3.  Bound as above"""
    ctx = binding.Context()
    X = (of_x * torch.randn(n, d, device="cuda")).bfloat16()
    S0 = of_s0 * torch.randn(d, 1, device="cuda")
    B = torch.empty(d, 1, device="cuda")
    L = binding.make_layer(torch.empty(16, d, device="cuda", dtype=torch.bfloat16), X, 1)
    ctx.basis(L, X, K, 3, S0, 0, B)
    ctx.check()
    q = S0.double() / S0.double().norm()
    for _ in range(K):
        q = X.double().T @ (X.double() @ q)
        q = q / q.norm()
    assert (B.double() - q).norm() <= (K + 1) * 4e-6


@pytest.mark.parametrize("e", [-54, -40, 40, 50])
def test_powers_of_two_give_the_same_bits(e):
    """every rounding of a basis scales with a power of two"""
    ctx = binding.Context()
    n, d = 300, 1032
    X = torch.randn(n, d, device="cuda").bfloat16()
    L = binding.make_layer(torch.empty(16, d, device="cuda", dtype=torch.bfloat16), X, 1)
    got = torch.empty(2, d, 1, device="cuda")
    ctx.basis(L, X, 3, 3, None, 0, got[0])
    ctx.basis(L, X * 2.0 ** e, 3, 3, None, 0, got[1])
    ctx.check()
    assert torch.equal(got[0], got[1])


def test_zero_column_is_reported():
    ctx = binding.Context()
    X = torch.randn(100, 64, device="cuda").bfloat16()
    B = torch.empty(64, 1, device="cuda")
    L = binding.make_layer(torch.empty(16, 64, device="cuda", dtype=torch.bfloat16), X, 1)
    ctx.basis(L, X, 0, 3, torch.zeros(64, 1, device="cuda"), 0, B)
    with pytest.raises(binding.AgzoError):
        ctx.check()
    ctx.basis(L, X, 2, 3, torch.zeros(64, 1, device="cuda"), 0, B)
    with pytest.raises(binding.AgzoError):
        ctx.check()
    ctx.basis(L, X, 2, 3, None, 0, B)
    ctx.check()


def _launches(ctx, call):
    call()
    ctx.stream.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=ctx.stream):
        call()
    n = ctypes.c_size_t(0)
    assert binding.load().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("seed", [3, 11])
def test_no_planes_where_the_column_is_read(seed):
    """a power sketch, and the feature-space start of a basis, of few tokens: a launch less than of many, whose products read planes; and
    the start's result against fp64, beside a layer that does read them"""
    ctx = binding.Context(stream=torch.cuda.Stream())
    few, many = (torch.randn(n, 264, device="cuda").bfloat16() for n in (8191, 8192))
    q, s = torch.randn(264, 1, device="cuda"), torch.empty(264, 1, device="cuda")
    b = torch.empty(2, 264, 1, device="cuda")
    q0 = torch.empty(264, 1, device="cuda")
    lay = [binding.make_layer(torch.empty(16, 264, device="cuda", dtype=torch.bfloat16), x, 1) for x in (few, many)]
    torch.cuda.synchronize()
    with torch.cuda.stream(ctx.stream):
        sketch = [_launches(ctx, lambda: ctx.layer_forward_sketch(l, None, x, None, binding.SKETCH_POWER, q, 0, s, None, None)) for l, x in zip(lay, (few, many))]
        basis = [_launches(ctx, lambda: ctx.basis(l, x, 1, seed, None, binding.INIT_FEATURE, o)) for l, x, o in zip(lay, (few, many), b)]
        assert sketch[0] == sketch[1] - 1
        assert basis[0] == basis[1] - 2                # (and one that the projection saves by normalising its result)
        ctx.basis_many([(l, x, seed, None, o) for l, x, o in zip(lay, (few, many), b)], 2, binding.INIT_FEATURE)
        ctx.fill_normal(q0, seed, binding.TAG_Q0)
        ctx.check()
    for x, o in zip((few, many), b):
        y = q0.double()
        for _ in range(3):
            y = x.double().T @ (x.double() @ y)
            y = y / y.norm()
        assert (o.double() - y).norm() <= 4 * 4e-6
    ctx.close()
