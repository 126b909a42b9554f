"""fb_fold_batch at its edges: pieces and remainders of the batch loop, sizes and addresses that rule out
16-byte pieces, both forms of the batch split, one and two tensors.  Against float64 sums: the fp32 sum of B
values is off by at most (B - 1) 2^-24 sum |x|, and a bf16 result (8 significant bits) is rounded once more:
half of its last place, at most 2^-8 of itself."""
import pytest
import torch

from paper_2505_12044_amd import api

pytestmark = pytest.mark.gpu


def _check(g, got):
    x = g.double()
    ref, mag = x.sum(0, keepdim=True), x.abs().sum(0, keepdim=True)
    bound = (g.shape[0] - 1) * 2.0 ** -24 * mag
    if g.dtype == torch.bfloat16:
        bound = bound + 2.0 ** -8 * (ref.abs() + bound)
    err = (got.double() - ref).abs()
    assert got.shape == ref.shape and got.dtype == g.dtype
    assert bool((err <= bound).all()), float((err - bound).max())


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B", [1, 2, 3, 4, 7, 16, 47, 200])
@pytest.mark.parametrize("n0,n1", [(1, 0), (7, 8), (8, 4096 + 8), (1000, 1002), (12 * 333, 12 * 65)])
def test_fold_batch(dtype, B, n0, n1):
    gen = torch.Generator(device="cuda").manual_seed(B * 10007 + n0 + n1)
    gs = [torch.randn((B, n), generator=gen, device="cuda").to(dtype) for n in (n0, n1) if n]
    got = api.fb_fold_batch(*gs)
    torch.cuda.synchronize()
    for g, r in zip(gs, got):
        _check(g, r)


@pytest.mark.parametrize("dtype,n", [(torch.bfloat16, 2_200_000), (torch.float32, 1_050_001)])
def test_fold_batch_unsplit(dtype, n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    g = torch.randn((13, n), generator=gen, device="cuda").to(dtype)
    got = api.fb_fold_batch(g)
    torch.cuda.synchronize()
    _check(g, got[0])


def test_fold_batch_unaligned_rows():
    g = torch.randn(5 * 64 + 1, device="cuda").to(torch.bfloat16)[1:].view(5, 64)      # contiguous, 2-byte aligned
    got = api.fb_fold_batch(g)
    torch.cuda.synchronize()
    _check(g, got[0])


def test_fold_batch_in_several_launches():
    # 2^32 + 1 values: one by one (the rows are not 16-byte aligned) they are more threads than one launch takes
    n = (1 << 32) + 1
    g = torch.ones((2, n), dtype=torch.bfloat16, device="cuda")
    g[1, ::4097] = 3.0
    g[0, -1] = 5.0
    got, = api.fb_fold_batch(g)
    g[0] += g[1]
    assert got.shape == (1, n) and torch.equal(got[0], g[0])
