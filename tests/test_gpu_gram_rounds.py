"""Gram matrices of head counts that do not divide the compute units: a head gets as many workgroups as all hold at once, and where
their sums are longer than those of the rounded-up number each is made of two (7 x 4 and 100 heads, and the last four shapes).  Against float64.

A wavefront adds at most 8 products (of 2 tokens; 16-bit: one of 16) per chunk of 16 tokens to a sum, each addition off by at most
2^-23 of it (the 16-bit matrix cores truncate), and the sums of a diagonal entry only grow: the bound, which holds for the
other entries relative to the diagonal."""
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("heads,qpk,n", [(7, 4, 5001), (20, 1, 2000), (48, 2, 1111), (100, 1, 2100), (127, 3, 333),
                                         (13, 4, 8192), (20, 4, 2000), (48, 4, 1111), (127, 4, 333)])
def test_head_counts_that_do_not_divide_the_device(dtype, heads, qpk, n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn(heads * qpk, n, 128, device="cuda", generator=gen).to(dtype)
    got = squat.build_subspace(q, qpk, 0, want_gram=True)[2].double()
    per_head = 256 // heads
    units = qpk * -(-n // 16)
    chunks = -(-units // (4 * per_head)) + 4
    if min(-(-units // 32), -(-256 // heads)) > per_head:
        chunks = chunks // 2 + 4
    bound = chunks * (8 if dtype == torch.float32 else 1) * 2.0 ** -23
    for h in range(heads):
        x = q[h * qpk:(h + 1) * qpk].reshape(-1, 128).double()
        want = x.T @ x
        d = want.diagonal().sqrt()
        assert ((got[h] - want).abs() / (d[:, None] * d[None, :])).max().item() <= bound
        assert torch.equal(got[h], got[h].T)
