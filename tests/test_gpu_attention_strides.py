"""The attention core on rows of wider tensors: whole and partial tiles of keys, the same bits as from contiguous ones."""
import pytest
import torch

from launches import kernels
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,T,H,Hkv", [(3, 64, 2, 1), (2, 150, 6, 3), (1, 17, 1, 1)])
def test_strided_rows(n_seq, T, H, Hkv):
    g = torch.Generator(device="cuda").manual_seed(T)
    n, ctx = n_seq * T, binding.Context()
    q, k, v = (torch.randn(n, w * 128, device="cuda", generator=g).bfloat16() for w in (H, Hkv, Hkv))

    def wide(x, before, behind):      # the same values in rows with NaN on either side
        buf = torch.full((n, before + x.shape[1] + behind), float("nan"), device="cuda", dtype=torch.bfloat16)
        return buf[:, before:before + x.shape[1]].copy_(x)
    want, got = torch.empty_like(q), wide(torch.zeros_like(q), 24, 8)
    ctx.glue_attention(q, k, v, want, n_seq, T)
    ctx.glue_attention(wide(q, 8, 0), wide(k, 0, 16), wide(v, 40, 8), got, n_seq, T)
    ctx.check()
    assert torch.isfinite(want).all() and torch.equal(got, want)
    assert torch.isnan(got._base[:, :24]).all() and torch.isnan(got._base[:, 24 + q.shape[1]:]).all()


# name: (q, k, v, out) as (first row, first column) in one buffer, tokens H 128 + 2 Hkv 128 + 64 wide, or contiguous tensors by name
@pytest.mark.parametrize("n_seq,T,H,Hkv", [(2, 150, 4, 4), (3, 64, 2, 1), (1, 300, 6, 3)])
def test_out_may_overlap_its_inputs(n_seq, T, H, Hkv):
    """the bits of a call whose tensors are apart, whatever `out` lies in: replaced row by row, a row or some columns further on, in rows of another
    length"""
    g = torch.Generator(device="cuda").manual_seed(T)
    n, ctx, dq, dk = n_seq * T, binding.Context(), H * 128, Hkv * 128
    q, k, v = (torch.randn(n, w, device="cuda", generator=g).bfloat16() for w in (dq, dk, dk))
    want = torch.empty_like(q)
    ctx.glue_attention(q, k, v, want, n_seq, T)
    width = dq + 2 * dk + 64

    def placed(cols, out_at, out_ld=width):
        """views of q, k, v at the columns `cols` of one buffer and of `out` at its element out_at"""
        buf = torch.zeros((n + 2) * width + dq, device="cuda", dtype=torch.bfloat16)
        tens = [torch.as_strided(buf, x.shape, (width, 1), c).copy_(x) for x, c in zip((q, k, v), cols)]
        return (*tens, torch.as_strided(buf, q.shape, (out_ld, 1), out_at))
    cols = (0, dq, dq + dk)
    cases = {"q": placed(cols, 0), "beside": placed((64, dq + 64, dq + dk + 64), 64), "q, columns further": placed(cols, 8), "q, a row further": placed(cols, width),
             "k and v": placed(cols, dq), "v": placed((0, dq, dq + dk), dq + dk), "rows of another length": placed(cols, 0, width - 64)}
    for name, (a, b, c, out) in cases.items():
        ctx.glue_attention(a, b, c, out, n_seq, T)
        ctx.check()
        assert torch.equal(out, want), name
    # contiguous: v itself, and q a row back
    if H == Hkv:
        vv = v.clone()
        ctx.glue_attention(q, k, vv, vv, n_seq, T)
        assert torch.equal(vv, want)
    flat = torch.empty(n + 1, dq, device="cuda", dtype=torch.bfloat16)
    flat[1:] = q
    ctx.glue_attention(flat[1:], k, v, flat[:n], n_seq, T)
    assert torch.equal(flat[:n], want)
    qq = q.clone()
    ctx.glue_attention(qq, k, v, qq, n_seq, T)
    ctx.check()
    assert torch.equal(qq, want)


@pytest.mark.parametrize("at,copies", [(0, 0), (768, 0), (8, 1), (640, 1)])
def test_copies_only_what_out_lies_in(at, copies):
    """columns of one buffer: in place of q and beside all inputs nothing is copied, across q's columns q is, across v's v"""
    buf, stream = torch.randn(100, 1024, device="cuda").bfloat16(), torch.cuda.Stream()
    ctx = binding.Context(stream)
    q, k, v, out = (buf[:, a:b] for a, b in ((0, 256), (256, 384), (512, 640) if at != 640 else (768, 896), (at, at + 256)))

    def call():
        ctx.glue_attention(q, k, v, out, 2, 50)
    torch.cuda.synchronize()
    call()
    ctx.check()
    names, _ = kernels(stream, call)
    assert sum("glue_copy_rows" in s for s in names) == copies, names
