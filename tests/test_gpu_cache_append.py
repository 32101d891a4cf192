"""The fused launches of the cache: one per appended token (key copy, value eviction with its quantization, value copy)
and one per logits call (packed and full-precision keys).

The evicted values must be stored exactly as squat_quantize_keys(update = NULL) stores them - both run the same
arithmetic - for every group size and type, with constant groups, groups whose zero-point is large against the step (the
written-out form with the clamp), steps below the normal fp16 range and infinities among them.  The residual logits are
fp32 dot products of 128 terms: off by at most 128 * 2^-24 < 1e-5 of sum |q_c k_c|."""
import numpy as np
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu

D = 128
DT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}


def _values(b, h, n, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(77)
    v = torch.randn((b, h, n, D), generator=g, device="cuda")
    v[:, :, 1] = 3.0                                     # constant
    v[:, :, 2] = 1000.0 + 0.5 * v[:, :, 2]               # zero-point large against the step
    v[:, :, 3] *= 1e-6                                   # step below the normal fp16 numbers
    v[:, :, 4, 32:64] = 0.0                              # one constant group beside ordinary ones
    v[:, :, 5, 7] = float("inf")
    v[:, :, 6, :64] *= 1e4
    return v.to(dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("bits,group", [(2, 32), (2, 64), (2, 128), (4, 32), (4, 64), (4, 128)])
def test_evicted_values_are_stored_as_quantize_keys_stores_them(bits, group, dtype):
    b, h, r, n = 3, 5, 4, 20                             # 15 heads: a workgroup that is not full
    v = _values(b, h, n, DT[dtype])
    cache = squat.Cache(b, h, 2, bits, group, 128, r, 32, DT[dtype], None, True)
    cache.prefill(v[:, :, :2], v[:, :, :2])
    for t in range(2, n):
        cache.append(v[:, :, t], v[:, :, t])
    cnt, st = cache.counts(), cache.stores()
    assert cnt.values_quantized == n - r and cnt.values_residual == r
    # token by token: a call's tiles choose between two forms of the arithmetic, a tile of one token as that token needs
    per_token = [squat.quantize_keys(v[:, :, t:t + 1], None, bits, group, 128) for t in range(n - r)]
    want = [torch.cat([p[i] for p in per_token], 2) for i in range(3)]
    torch.cuda.synchronize()
    for name, w in zip(("codes", "scale", "zero"), want):
        got = st["value_" + name][:, :, :n - r]
        assert torch.equal(got.view(torch.int16 if name != "codes" else torch.int32),
                           w.view(torch.int16 if name != "codes" else torch.int32)), name
    ring = st["value_residual"]
    for i in range(r):
        assert torch.equal(ring[:, :, (cnt.value_ring_head + i) % r], v[:, :, n - r + i])
    keys = st["key_residual"][:, :, :cnt.keys_residual]
    assert torch.equal(keys, v[:, :, n - cnt.keys_residual:])


@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("qdt", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("n,r", [(1, 32), (31, 32), (32, 32), (33, 32), (160, 128), (255, 128), (95, 96), (1023, 1024)])
def test_logits_of_the_full_precision_tail(n, r, qdt, per_channel):
    b, h, qpk, kdt = 2, 3, 5, torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    k = torch.randn((b, h, n, D), generator=g, device="cuda").to(kdt)
    q = torch.randn((b, h * qpk, D), generator=g, device="cuda").to(DT[qdt])
    cache = squat.Cache(b, h, qpk, 2, 32, 32, r, 1024 // r * r, kdt, None, False, key_per_channel=per_channel)
    cache.prefill(k)
    out = torch.full((b, h * qpk, n + 8), -5.0, device="cuda")
    cache.key_scores(q, 0.5, out=out)
    cnt = cache.counts()
    nq = cnt.keys_quantized
    assert nq == n // r * r
    tail = k[:, :, nq:].double().cpu().numpy()
    qd = q.double().cpu().numpy().reshape(b, h, qpk, D)
    got = out.double().cpu().numpy().reshape(b, h, qpk, n + 8)
    want = 0.5 * (qd @ tail.transpose(0, 1, 3, 2))
    bound = 0.5 * (np.abs(qd) @ np.abs(tail).transpose(0, 1, 3, 2))
    assert np.all(np.abs(got[..., nq:n] - want) <= 1e-5 * bound)
    assert (got[..., n:] == -5.0).all() and (got[..., :n] != -5.0).all()


# Full-precision keys beside packed ones share their launch up to 24 MiB (in whole eights per head): below, on and above
# that line; the packed keys in one and in several grid layers (z); full-precision keys alone.
@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("b,h,n,launches", [(1, 3, 1000, 1), (5, 40, 550, 1), (64, 40, 40, 1), (1536, 8, 40, 1),
                                            (1536, 8, 41, 2), (12289, 1, 33, 2), (32768, 1, 33, 2), (1, 32771, 33, 2),
                                            (35000, 2, 33, 2), (32767, 3, 33, 2), (32768, 1, 2, 1), (1, 65537, 2, 1)])
def test_full_precision_tail_of_many_heads(b, h, n, launches, per_channel):
    packed, eights = n // 32 * 32, (n % 32 + 7) // 8
    assert launches == 1 + (packed > 0 and b * h * eights * 8 * 256 > 24 << 20)      # (test_logits_grids.py sees them)
    g = torch.Generator(device="cuda")
    g.manual_seed(b + h)
    k = torch.randn((b, h, n, D), generator=g, device="cuda", dtype=torch.bfloat16)
    q = torch.randn((b, h, D), generator=g, device="cuda", dtype=torch.bfloat16)
    cache = squat.Cache(b, h, 1, 2, 32, 32, 32, (n + 31) // 32 * 32, torch.bfloat16, None, False, key_per_channel=per_channel)
    cache.prefill(k)
    out = torch.full((b, h, n + 1), -5.0, device="cuda")
    cache.key_scores(q, 1.0, out=out)
    nq = n // 32 * 32
    if nq:
        st = [cache.stores()["key_" + i] for i in ("codes", "scale", "zero")]
        st = [x[:, :, :nq].contiguous() if not per_channel else x[:, :, :nq // 32].contiguous() for x in st]
        want = squat.key_scores_per_channel(q, *st, 2, 1) if per_channel else squat.key_scores(q, *st, 2, 32, 1)
        assert torch.equal(out[:, :, :nq], want)
    prod = q.float()[:, :, None] * k[:, :, nq:].float()
    err = (out[:, :, nq:n].double() - prod.double().sum(-1)).abs()
    assert bool((err <= 1e-5 * prod.abs().double().sum(-1)).all())
    assert bool((out[:, :, n] == -5.0).all())
