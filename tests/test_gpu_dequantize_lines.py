"""Dequantized keys bit for bit: every width, grouping and output type, outputs on both sides of the 4 MB from which they are streamed,
odd token counts, and rows with room between them, which stays untouched.  code * scale + zero is exact in float64 and rounded once to
float32, then to the output type."""
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu


def _check(call, codes, scale, zero, want, bits, group, dtype):
    b, h, n, d = want.shape
    room = torch.full((b, h, n, d + 8), 7.0, dtype=dtype, device="cuda")
    call(codes, scale, zero, bits, group, out=room[..., :d])
    want = want.float().to(dtype)
    assert torch.equal(room[..., :d], want) and (room[..., d:] == 7.0).all()
    assert torch.equal(call(codes, scale, zero, bits, group, dtype), want)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("heads,n", [(3, 1), (3, 37), (5, 3333)])
def test_per_token(dtype, bits, heads, n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    for group in (32, 64, 128):
        words = torch.randint(-2 ** 31, 2 ** 31, (2, heads, n, 4 * bits), device="cuda", generator=gen, dtype=torch.int64).to(torch.int32)
        scale = torch.rand(2, heads, n, 128 // group, device="cuda", generator=gen).half()
        zero = torch.randn(2, heads, n, 128 // group, device="cuda", generator=gen).half()
        sh = bits * torch.arange(32 // bits, device="cuda")
        c = ((words.to(torch.int64)[..., None] >> sh) & (2 ** bits - 1)).flatten(-2).double()
        want = c * scale.double().repeat_interleave(group, -1) + zero.double().repeat_interleave(group, -1)
        _check(squat.dequantize_keys, words, scale, zero, want, bits, group, dtype)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("heads,n", [(3, 32), (3, 160), (5, 3328)])
def test_per_channel(dtype, bits, heads, n):
    gen = torch.Generator(device="cuda").manual_seed(n + 1)
    words = torch.randint(-2 ** 31, 2 ** 31, (2, heads, n // 32, 128, bits), device="cuda", generator=gen, dtype=torch.int64).to(torch.int32)
    scale = torch.rand(2, heads, n // 32, 128, device="cuda", generator=gen).half()
    zero = torch.randn(2, heads, n // 32, 128, device="cuda", generator=gen).half()
    sh = bits * torch.arange(32 // bits, device="cuda")
    c = ((words.to(torch.int64)[..., None] >> sh) & (2 ** bits - 1)).flatten(-2).transpose(-1, -2).flatten(-3, -2).double()
    want = c * scale.double().repeat_interleave(32, -2) + zero.double().repeat_interleave(32, -2)
    _check(squat.dequantize_keys_per_channel, words, scale, zero, want, bits, 32, dtype)
