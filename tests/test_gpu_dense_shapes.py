"""The dense Gaussian sweep at the edges of its work split: rows in pairs, four columns a thread, vector and scalar accesses."""
import pytest
import torch

from paper_2601_17261_amd import binding

pytestmark = pytest.mark.gpu
TAG_DENSE = 3


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols,pad", [(1, 1, 0), (1, 4, 0), (1, 1027, 0), (2, 8, 4), (3, 4, 0), (5, 1024, 8), (7, 130, 1), (256, 3, 5), (1025, 516, 0)])
def test_against_the_generator(rows, cols, pad, dtype):
    """theta + c z, rounded once: the sum in fp64 rounds to the same value except where fp32 rounds on the way (one unit in the last
    place of fp32, and a value of bf16 at a tie of that size)"""
    ctx = binding.Context()
    whole = torch.randn(rows, cols + pad, device="cuda").to(dtype)
    theta, before = whole[:, :cols], whole.clone()
    z = torch.empty(rows, cols, device="cuda")
    ctx.fill_normal(z, 77, TAG_DENSE)
    c = torch.tensor(0.37, device="cuda").item()
    g = torch.tensor([1.5], dtype=torch.float64, device="cuda")
    ctx.dense_perturb(theta, 77, c, g)
    ctx.check()
    want = before[:, :cols].double() + float(torch.tensor(c * 1.5, dtype=torch.float32)) * z.double()
    assert torch.equal(whole[:, cols:], before[:, cols:])
    half_ulp = want.abs() * (2.0 ** -24 if dtype == torch.float32 else 2.0 ** -8)      # 24 and 8 significant bits
    assert ((theta.double() - want).abs() <= half_ulp * 1.01 + 2.0 ** -24 * (want.abs() + 1e-30)).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(2731, 2929), (2731, 2930), (8000001, 1), (3, 2666667)])
def test_large_blocks_of_odd_rows(rows, cols, dtype):
    """on both sides of the size from which a thread takes two rows: the bound of the test above"""
    ctx = binding.Context()
    theta = torch.randn(rows, cols, device="cuda").to(dtype)
    z = torch.empty(rows, cols, device="cuda")
    ctx.fill_normal(z, 5, TAG_DENSE)
    c = torch.tensor(0.25, device="cuda").item()
    want = torch.addcmul(theta.double(), z.double(), torch.full_like(z, c, dtype=torch.float64))
    ctx.dense_perturb(theta, 5, c)
    ctx.check()
    half_ulp = want.abs() * (2.0 ** -24 if dtype == torch.float32 else 2.0 ** -8)
    assert ((theta.double() - want).abs() <= half_ulp * 1.01 + 2.0 ** -24 * (want.abs() + 1e-30)).all()
