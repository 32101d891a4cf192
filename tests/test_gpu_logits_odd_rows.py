"""Per-token stores whose rows (scales of one head) start at a multiple of 4 bytes only, or of 2: whole units of 16 tokens are
fetched with 16-byte loads in both cases.  Bounds as derived in test_gpu_scores.py
(4e-5 of sum_c |q_c| (step code_c + |zero|), the two parts that are summed apart) and, for the rotary form without a
turn (inv_freq = 0), 2e-3 of the same sum (four roundings to fp16)."""
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("n", [15, 33, 47, 66, 1001, 1030])
@pytest.mark.parametrize("bits,group", [(2, 32), (4, 32), (2, 64), (4, 64), (2, 128), (4, 128)])
def test_rows_at_any_offset(bits, group, n, rope):
    b, h, qpk = 2, 3, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(n + bits + group)
    codes = torch.randint(-2 ** 31, 2 ** 31 - 1, (b, h, n, 4 * bits), generator=g, device="cuda", dtype=torch.int32)
    scale = torch.rand((b, h, n, 128 // group), generator=g, device="cuda").half()
    zero = torch.randn((b, h, n, 128 // group), generator=g, device="cuda").half()
    q = torch.randn((b, h * qpk, 128), generator=g, device="cuda").to(torch.bfloat16)
    per = 32 // bits
    shift = bits * torch.arange(per, device="cuda")
    c = ((codes.long()[..., None] >> shift) & (2 ** bits - 1)).reshape(b, h, n, 128).double()
    step, zp = scale.double().repeat_interleave(group, -1), zero.double().repeat_interleave(group, -1)
    deq, size = c * step + zp, c * step + zp.abs()
    if rope:
        got = squat.key_scores_rope(q, codes, scale, zero, bits, group, qpk, torch.zeros(64, device="cuda"))
    else:
        got = squat.key_scores(q, codes, scale, zero, bits, group, qpk)
    qd = q.double().reshape(b, h, qpk, 1, 128)
    want = (qd * deq[:, :, None]).sum(-1).reshape(b, h * qpk, n)
    bound = (qd.abs() * size[:, :, None]).sum(-1).reshape(b, h * qpk, n)
    assert bool(((got.double() - want).abs() <= (2e-3 if rope else 4e-5) * bound).all())
