"""The attention core around its tiles: a key more or fewer than 64, queries of the last wave only, head counts that the
four heads of a preparation group do not divide.  Oracle, tolerances and the causality check of test_gpu_decoder.py."""
import pytest
import torch

import test_gpu_decoder
from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,T,H,Hkv", [(2, 63, 1, 1), (1, 65, 6, 3), (1, 97, 2, 2), (1, 321, 5, 1)])
def test_attention_core(n_seq, T, H, Hkv):
    test_gpu_decoder.test_attention_core_matches_oracle(binding.Context(), n_seq, T, H, Hkv)


@pytest.mark.parametrize("at", [40, 104, 160, 201])
def test_values_behind_a_queries_group_do_not_reach_it(at):
    """An infinite value at token `at` stays out of every output before its group of 32 tokens: later keys are no part of those
    sums.  (Inside the group its probability is 0 for the earlier queries, and 0 x inf is NaN.)"""
    T, H = 202, 3
    ctx = binding.Context()
    q, k, v = (torch.randn(T, w * 128, device="cuda").bfloat16() for w in (H, 1, 1))
    want, got, v2 = torch.empty_like(q), torch.empty_like(q), v.clone()
    v2[at] = float("inf")
    ctx.glue_attention(q, k, v, want, 1, T)
    ctx.glue_attention(q, k, v2, got, 1, T)
    ctx.check()
    first = at // 32 * 32
    assert torch.equal(got[:first], want[:first]) and not torch.isfinite(got[at:]).any()


@pytest.mark.parametrize("T,H", [(97, 2), (202, 3), (515, 1)])
def test_probabilities_are_rounded_around_the_maximum_of_32_keys_at_a_time(T, H):
    """The steps of the online softmax in 64 bits, with the one rounding that the kernel makes in them (probabilities to bf16):
    what is left is the rounding of the output, except where the fp32 arithmetic of queries, keys and probabilities falls on the
    other side of a rounding, some 1e-4 of them each.  Around other maxima every probability rounds differently, and 9 to 17 %
    of the outputs with them (64 keys at a time)."""
    ctx = binding.Context()
    g = torch.Generator(device="cuda").manual_seed(T)
    q, k, v = (torch.randn(T, w * 128, device="cuda", generator=g).bfloat16() for w in (H, 1, 1))
    out = torch.empty_like(q)
    ctx.glue_attention(q, k, v, out, 1, T)
    ctx.check()
    angle = torch.arange(T, device="cuda").double()[:, None] * 1e6 ** (-torch.arange(64, device="cuda").double() / 64)

    def prepared(x):
        x = x.double()
        x = x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6)
        a, b = x[:, :64], x[:, 64:]
        return torch.cat((a * angle.cos() - b * angle.sin(), b * angle.cos() + a * angle.sin()), -1).bfloat16().double()
    K, V, pos = prepared(k), v.double(), torch.arange(T, device="cuda")
    wrong = 0
    for h in range(H):
        S = prepared(q[:, 128 * h:128 * h + 128]) @ K.T / (128 ** 0.5 * torch.log(torch.tensor(2.0, dtype=torch.float64)).item())
        S.masked_fill_(pos[None, :] > pos[:, None], float("-inf"))
        m, l, acc = torch.full((T, 1), float("-inf"), device="cuda", dtype=torch.float64), 0.0, 0.0
        for kb in range(0, T, 32):
            s = S[:, kb:kb + 32]
            new = torch.maximum(m, s.max(1, keepdim=True).values)
            p, alpha = torch.exp2(s - new), torch.exp2(m - new)
            l, acc, m = l * alpha + p.sum(1, keepdim=True), acc * alpha + p.bfloat16().double() @ V[kb:kb + 32], new
        wrong += (out[:, 128 * h:128 * h + 128] != (acc / l).bfloat16()).sum().item()
    assert wrong < 0.03 * out.numel(), wrong / out.numel()
