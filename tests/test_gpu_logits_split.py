"""The logits kernels share a sequence among more or fewer wavefronts depending on how many sequences a launch holds:
a few sequences are spread over the chip down to one pair of 16-token units (one step, one epoch) a wavefront, many
keep long ranges per wavefront.  Both ends of that rule on the same store, at token counts around the units, pairs,
epochs and slabs: a launch of one sequence against the float64 oracle, and a launch of 600 copies of it, whose copies
must agree with each other bit for bit and with the oracle.

Bounds: as derived in test_gpu_scores.py (4e-5 of sum_c |q_c| |deq_c|: fp32 sums), test_gpu_scores_pc.py (the same plus
fp16 operands normalised by the largest |q| and the largest step of a token group) and test_gpu_scores_rope.py (2e-3
of the rotary-pair sum: four roundings to fp16)."""
import numpy as np
import pytest
import torch

from oracle import squat_oracle as O
from paper_2503_24358_amd import squat, synth
from tests import util

pytestmark = pytest.mark.gpu

H, QPK, POS0, SCALE = 2, 4, 7, 0.25
COPIES = 600
INV_FREQ = (10000.0 ** (-np.arange(64) / 64.0)).astype(np.float32)


def _store(n, bits, axis):
    x = synth.keys(9100 + n + bits, H, n, batch=1)[0].astype(np.float64)
    outs = [O.quantize_keys(x[h], None, bits, 32, 128, **({} if axis == "token" else {"axis": "channel"}))
            for h in range(H)]
    return tuple(np.stack([o[k] for o in outs]) for k in ("codes", "scale", "zero"))


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("axis,bits,n", [("token", 2, 1), ("token", 2, 33), ("token", 4, 120), ("token", 2, 333),
                                         ("token", 4, 1000), ("token", 2, 4111), ("channel", 2, 32), ("channel", 4, 96),
                                         ("channel", 2, 544), ("channel", 4, 1056), ("channel", 2, 4160)])
def test_logits_of_one_and_of_many_sequences(axis, bits, n, rope):
    codes, scale, zero = _store(n, bits, axis)
    words = O.pack_codes(codes, bits) if axis == "token" else O.pack_codes_tokens(codes, bits)
    dev = [torch.from_numpy(a).cuda()[None] for a in (words.view(np.int32), scale, zero)]
    q32 = synth.rng(9200 + n).standard_normal((1, H * QPK, 128)).astype(np.float32)
    qraw, qval = synth.store(q32, synth.BF16)
    q = util.to_device(qraw, synth.BF16)
    inv = torch.from_numpy(INV_FREQ).cuda()

    def logits(copies):
        a = [t.repeat(copies, *([1] * (t.dim() - 1))) for t in dev]
        qq = q.repeat(copies, 1, 1)
        if axis == "token":
            if rope:
                return squat.key_scores_rope(qq, *a, bits, 32, QPK, inv, POS0, SCALE)
            return squat.key_scores(qq, *a, bits, 32, QPK, SCALE)
        if rope:
            return squat.key_scores_rope_per_channel(qq, *a, bits, QPK, inv, POS0, SCALE)
        return squat.key_scores_per_channel(qq, *a, bits, QPK, SCALE)

    one, many = logits(1), logits(COPIES)
    torch.cuda.synchronize()
    assert torch.equal(many, many[:1].expand_as(many)), "copies of one sequence differ inside a launch"
    for got in (one[0].cpu().numpy().astype(np.float64), many[0].cpu().numpy().astype(np.float64)):
        for hq in range(H * QPK):
            h = hq // QPK
            kw = {} if axis == "token" else {"axis": "channel"}
            khat = O.dequantize_keys(codes[h], scale[h], zero[h], 32, **kw)
            qv = qval[0, hq]
            if rope:
                want = O.key_scores_rope(qv[None], codes[h], scale[h], zero[h], 32, INV_FREQ, POS0, SCALE, **kw)[0]
                rho = np.sqrt(khat[:, :64] ** 2 + khat[:, 64:] ** 2)
                bound = 2e-3 * SCALE * (rho @ (np.abs(qv[:64]) + np.abs(qv[64:])))
            else:
                want = O.key_scores(qv[None], codes[h], scale[h], zero[h], 32, SCALE, **kw)[0]
                bound = 4e-5 * SCALE * (np.abs(khat) @ np.abs(qv))
                if axis == "channel":
                    qmax = np.abs(qval[0, h * QPK:(h + 1) * QPK]).max()
                    dmax = np.repeat(scale[h].astype(np.float64).max(axis=1), 32)
                    bound = bound + SCALE * 128 * (2 ** bits - 1) * 2.0 ** -24 * qmax * dmax
            assert np.all(np.abs(got[hq] - want) <= bound + 1e-30), (hq, float(np.abs(got[hq] - want).max()))
