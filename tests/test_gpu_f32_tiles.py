"""fp32 forwards in both tile sizes, at the edges of either and around the number of tiles that decides: losses and outputs from fp64
accumulators, so they agree with fp64 to its rounding (losses) and to one rounding to fp32 (outputs)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import agzo as oagzo
from paper_2601_17261_amd import binding, synth

pytestmark = pytest.mark.gpu
EPS, LR = float(np.float32(1e-3)), float(np.float32(1e-2))

# tokens, d_out, d_in, r: tiles of 32 (one, a row or column more, ranks past a slice, d_in below, at and past the slices in flight,
# rows that are not 16-byte vectors), 127 and 128 tiles of 64
SHAPES = [(32, 32, 32, 1), (33, 65, 31, 4), (64, 31, 129, 33), (100, 96, 160, 16), (1, 7, 5, 1), (95, 33, 257, 64), (127 * 64, 64, 36, 2), (8192, 61, 68, 3)]


@pytest.mark.parametrize("n,d_out,d_in,r", SHAPES)
def test_step_and_stored_output(n, d_out, d_in, r):
    r = min(r, n, d_in)
    ctx = binding.Context()
    W, X, T = synth.single_layer_problem(11, n, d_in, d_out, kind="rmsnorm", storage="f32")
    Wd, Xd, Td = (torch.from_numpy(a).cuda() for a in (W, X, T))
    Y = torch.empty(n, d_out, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    L = binding.make_layer(Wd, Xd, r, Y=Y)
    ctx.layer_forward_sketch(L, Wd, Xd, Y, binding.SKETCH_NONE, None, 0, None, binding.make_loss(Td), loss)
    ctx.check()
    want = X.astype(np.float64) @ W.astype(np.float64).T
    assert np.all(np.abs(Y.double().cpu().numpy() - want) <= 2.0 ** -24 * np.abs(want) + 1e-13 * np.abs(want).max())
    l0 = np.mean((want - T.astype(np.float64)) ** 2)
    assert abs(loss.item() - l0) <= 1e-12 * l0
    out = torch.zeros(2, 4, dtype=torch.float64, device="cuda")
    Ws = Wd.clone()
    ctx.step(binding.make_layer(Wd, Xd, r), Wd, Xd, binding.make_loss(Td), 1, EPS, LR, 5, 0, out[0])
    ctx.step(binding.make_layer(Ws, Xd, r), Ws, Xd, binding.make_loss(Td), 1, EPS, LR, 5, binding.SHARED_FORWARD, out[1])
    ctx.check()
    o = oagzo.agzo_step(W, X, T, r, 1, EPS, LR, 5, storage="f32")
    for got in out.cpu().numpy():
        assert abs(got[0] - o["L0"]) <= 1e-9 * o["L0"] and abs(got[1] - o["Lp"]) <= 1e-6 * o["Lp"]
        assert abs(got[3] - o["g"]) <= 2e-3 * abs(o["g"]) + 1e-9 * o["L0"] / EPS


# d_out, d_in of layers on 70 tokens (two or three tiles of 64 or 32, the last six wide) and 1100: tiles cut to one and to two blocks of 32,
# outputs past a block by one and short of it by one
EDGES = [(33, 64), (65, 36), (96, 129), (129, 31), (31, 160), (64, 200)]


def _set(shapes, tokens, r=8):
    got = []
    for i, (d_out, d_in) in enumerate(shapes):
        W, X, T = synth.single_layer_problem(20 + i, tokens, d_in, d_out, kind="rmsnorm", storage="f32")
        got.append(tuple(torch.from_numpy(a).cuda() for a in (W, X, T)))
    out = torch.zeros(len(got), 4, dtype=torch.float64, device="cuda")
    return got, out, [(binding.make_layer(w, x, r), w, x, binding.make_loss(t), 5 + i, out[i], None) for i, (w, x, t) in enumerate(got)]


@pytest.mark.parametrize("flags", [0, binding.SHARED_FORWARD])
@pytest.mark.parametrize("tokens", [70, 1100])
def test_a_layer_has_the_same_bits_in_every_launch(tokens, flags):
    """alone in 32 x 32 tiles, with layers of 400 tiles in 64 x 64 ones"""
    ctx = binding.Context()
    large = (64 * 13, 48)
    assert -(-1999 // 64) * 13 >= 400
    for shape in EDGES:
        (one,), out1, item1 = _set([shape], tokens)
        (two,), out2, item2 = _set([shape], tokens)
        _, out3, item3 = _set([large], 1999)
        w, x, t = one
        want = [((x.double() @ w.double().T - t.double()) ** 2).mean().item()]
        ctx.step_many(item1, 2, EPS, LR, flags)
        ctx.step_many(item2 + item3, 2, EPS, LR, flags)
        ctx.check()
        assert torch.equal(out1, out2) and torch.equal(one[0], two[0]), shape
        assert abs(out1[0, 0].item() - want[0]) <= 1e-12 * want[0]
    ctx.close()


def test_a_set_takes_one_launch():
    """layers above and below the line in one launch, where together they fill the chip"""
    ctx = binding.Context(stream=torch.cuda.Stream())

    def nodes(shapes):
        _, _, items = _set(shapes, 1000)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.stream(ctx.stream):
            ctx.step_many(items, 1, EPS, LR, 0)
            ctx.stream.synchronize()
            with torch.cuda.graph(graph, stream=ctx.stream):
                ctx.step_many(items, 1, EPS, LR, 0)
        n = ctypes.c_size_t(0)
        assert binding.load().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
        return n.value
    same = [(64 * 14, 256)] * 4          # 224 tiles each
    assert nodes(same[:2] + [(320, 256)] * 2) == nodes(same)
    ctx.check()
    ctx.close()
