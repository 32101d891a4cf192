"""Logits of sequences whose steps divide unevenly among wavefronts: every token is covered once, whatever the number of sequences
(each takes another number of workgroups) and the length (a last step that is not whole, fewer steps than wavefronts).  A sequence's
logits do not depend on how many others there are."""
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("qpk", [4, 8])
@pytest.mark.parametrize("heads,n", [(1, 32), (8, 4128), (9, 1632), (58, 2016), (150, 800), (257, 352), (320, 544), (600, 96), (1100, 64)])
@pytest.mark.parametrize("per_channel,rope", [(True, False), (True, True), (False, True), (False, False)])
def test_a_sequence_alone_and_among_others(per_channel, rope, heads, n, qpk):
    gen = torch.Generator(device="cuda").manual_seed(heads + n)
    words = torch.randint(-2 ** 31, 2 ** 31, (1, heads, n, 8), device="cuda", generator=gen, dtype=torch.int64).to(torch.int32)
    shape = (1, heads, n // 32, 128) if per_channel else (1, heads, n, 4)
    scale, zero = (torch.rand(shape, device="cuda", generator=gen).half() for _ in range(2))
    if per_channel:
        words = words.view(1, heads, n // 32, 128, 2)
    q = torch.randn(1, heads * qpk, 128, device="cuda", generator=gen).to(torch.bfloat16)
    freq = 10000.0 ** (-torch.arange(64, device="cuda") / 64.0)

    def logits(h0, h1):
        a = (q[:, h0 * qpk:h1 * qpk].contiguous(), *(x[:, h0:h1].contiguous() for x in (words, scale, zero)))
        out = torch.full((1, (h1 - h0) * qpk, n), float("nan"), device="cuda")
        if per_channel and rope:
            squat.key_scores_rope_per_channel(*a, 2, qpk, freq, 3, 0.1, out=out)
        elif per_channel:
            squat.key_scores_per_channel(*a, 2, qpk, 0.1, out=out)
        elif rope:
            squat.key_scores_rope(*a, 2, 32, qpk, freq, 3, 0.1, out=out)
        else:
            squat.key_scores(*a, 2, 32, qpk, 0.1, out=out)
        return out

    got = logits(0, heads)
    assert torch.isfinite(got).all()
    for h in {0, heads // 2, heads - 1}:
        want = logits(h, h + 1)
        # rotary: a wavefront's angles are advanced by the addition theorems from its own first epoch on (1e-6 of the largest logit)
        tol = 2e-5 * want.abs().max().item() if rope else 0.0
        assert (got[:, h * qpk:(h + 1) * qpk] - want).abs().max().item() <= tol
