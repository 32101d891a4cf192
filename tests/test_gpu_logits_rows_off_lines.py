"""Logits whose result rows begin on no 64-byte line (ordinary stores) against the same call into rows that do (non-temporal
stores): the same bits, nothing written outside a row's tokens, for every kernel and on both sides of the rule."""
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("b,h,qpk,n", [(1, 1, 1, 32), (2, 3, 4, 96), (2, 3, 8, 992), (16, 8, 4, 2496), (32, 8, 4, 2496), (64, 8, 4, 2496), (16, 8, 8, 1504), (3, 2, 5, 1504)])
def test_rows_on_and_off_the_lines_agree(b, h, qpk, n, per_channel, rope):
    g = torch.Generator(device="cuda")
    g.manual_seed(b + n)
    shape, meta = ((b, h, n // 32, 128, 2), (b, h, n // 32, 128)) if per_channel else ((b, h, n, 8), (b, h, n, 4))
    codes = torch.randint(-2 ** 31, 2 ** 31 - 1, shape, generator=g, device="cuda", dtype=torch.int32)
    scale = torch.rand(meta, generator=g, device="cuda").half()
    zero = torch.randn(meta, generator=g, device="cuda").half()
    q = torch.randn((b, h * qpk, 128), generator=g, device="cuda").half()
    inv = (10000.0 ** (-torch.arange(64) / 64.0)).float().cuda()
    out = []
    for width in (n + 16 - n % 16, n + 5):                      # rows a multiple of 64 bytes apart, and not
        buf = torch.full((b, h * qpk, width), 7.0, device="cuda")
        if per_channel and rope:
            squat.key_scores_rope_per_channel(q, codes, scale, zero, 2, qpk, inv, 3, 0.5, out=buf)
        elif per_channel:
            squat.key_scores_per_channel(q, codes, scale, zero, 2, qpk, 0.5, out=buf)
        elif rope:
            squat.key_scores_rope(q, codes, scale, zero, 2, 32, qpk, inv, 3, 0.5, out=buf)
        else:
            squat.key_scores(q, codes, scale, zero, 2, 32, qpk, 0.5, out=buf)
        assert bool((buf[:, :, n:] == 7.0).all())
        out.append(buf[:, :, :n])
    assert torch.equal(out[0], out[1])
