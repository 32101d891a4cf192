"""Gram matrices of launches on both sides of the rules that split the queries among workgroups (up to 16 workgroups, fp32
within and beyond one round, few or many heads) at token counts around a chunk of 16 and a workgroup's share of 32, 64
and 512 tokens, and (fp32, one head) of 7, 8, 9, 15, 16, 23, 24 and 31 partial matrices.

Bound: products of 16-bit queries are exact in fp32, those of fp32 queries and all sums are off by at most 2^-24 of the
running sum each, so an entry is within n 2^-24 sum |x y| (n = pooled tokens); accumulation chains are shorter than n,
and what is seen is a hundred times less."""
import numpy as np
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("heads,qpk,n", [(1, 1, 1), (1, 1, 15), (1, 1, 129), (1, 2, 512), (3, 1, 527), (8, 3, 33), (31, 1, 512),
                                         (32, 1, 100), (33, 1, 513), (40, 2, 300), (2, 1, 8209), (300, 1, 17),
                                         (16, 1, 512), (17, 1, 512), (24, 1, 200), (25, 1, 200), (28, 4, 1024), (48, 1, 2048),
                                         (1, 1, 896), (1, 1, 1010), (1, 1, 1152), (1, 1, 1920), (1, 1, 2048), (1, 1, 2941),
                                         (1, 1, 3072), (1, 1, 3968)])
def test_gram_matrix_of_any_split(heads, qpk, n, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(heads * 1000 + n)
    q = torch.randn((heads * qpk, n, 128), generator=g, device="cuda").to(dtype)
    _, _, gram = squat.build_subspace(q, qpk, 1, want_gram=True)
    torch.cuda.synchronize()
    x = q.double().cpu().numpy().reshape(heads, qpk * n, 128)
    got = gram.cpu().numpy().astype(np.float64)
    for h in {0, heads // 2, heads - 1}:
        want, mass = x[h].T @ x[h], np.abs(x[h]).T @ np.abs(x[h])
        assert np.all(np.abs(got[h] - want) <= (qpk * n + 1) * 2.0 ** -24 * mass)
        assert np.linalg.norm(got[h] - want) <= 1e-6 * np.linalg.norm(want)
        assert np.array_equal(got[h], got[h].T)
