"""The workloads this library is timed on: what a serving program asks of it, through the public calls of
paper_2503_24358_amd.squat, from one small head to a stack of 256.

A case is a dict of plain values; its "kind" names the call (or the chain of calls):

  subspace    prompt queries -> top-r directions, one layer or a stack of layers
  prepare     directions -> update matrix
  quantize    keys -> packed codes, scales, zero-points (a prompt, or a decode-time flush of the residual buffers)
  dequantize  packed store -> keys
  scores      attention logits of one decoded token per sequence, from the packed store
  path        the prefill of one layer: subspace, prepare, quantize
  cache       a short generation with the cache object: prefill, then append + logits for every token

Inputs are drawn on the GPU from the seed: queries that concentrate in a decaying set of directions, keys N(0, 1)
with 2 to 6 outlier channels per head (x8 to x15).  Update matrices and packed stores that a case takes as its input
are made here in plain torch, so that they do not depend on the library.  `exact` is the same computation in
64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2503_24358_amd import squat

D = 128
DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
DEV = "cuda:0"


# ---- cases ----------------------------------------------------------------------------------------------------- #

def listed():
    return [
        # the smallest prompt: one fp32 head of 512 tokens, the whole path (latency and launch count)
        {"name": "path_one_head", "kind": "path", "heads": 1, "qpk": 1, "n": 512, "keep": 0, "dtype": "f32", "r": 8,
         "lam": 1e-3, "bits": 2, "group": 32, "g": 32, "per_channel": False},
        # one multi-head layer of a 4096-token prompt, the newest 128 tokens kept in 16 bits
        {"name": "path_layer", "kind": "path", "heads": 32, "qpk": 1, "n": 4096, "keep": 128, "dtype": "bf16", "r": 16,
         "lam": 1e-3, "bits": 2, "group": 32, "g": 32, "per_channel": False},
        # one grouped-query layer of an 8192-token prompt: its subspace alone (layers arrive one by one in a prefill)
        {"name": "subspace_layer", "kind": "subspace", "heads": 8, "qpk": 4, "n": 8192, "dtype": "bf16", "r": 16},
        # all layers of a 32768-token prompt stacked on the head axis, the largest call
        {"name": "subspace_long", "kind": "subspace", "heads": 256, "qpk": 4, "n": 32768, "dtype": "bf16", "r": 32},
        # the update matrix at one of the paper's settings, the heads of one layer
        {"name": "prepare_layer", "kind": "prepare", "heads": 32, "r": 40, "lam": 1e-3, "g": 64, "full": False},
        # the prompt's keys, all layers stacked: the throughput case
        {"name": "quantize_long", "kind": "quantize", "batch": 1, "heads": 256, "n": 32768, "dtype": "bf16", "bits": 2,
         "group": 32, "g": 32, "per_channel": False, "update": True},
        # a decode-time flush: 64 sequences' residual buffers of 32 tokens, one layer
        {"name": "quantize_flush", "kind": "quantize", "batch": 64, "heads": 8, "n": 32, "dtype": "bf16", "bits": 2,
         "group": 32, "g": 32, "per_channel": False, "update": True},
        # the paper's own grouping (per channel), one layer of a long prompt in fp16, 4 bits, two blocks per key
        {"name": "quantize_channel", "kind": "quantize", "batch": 2, "heads": 8, "n": 8160, "dtype": "f16", "bits": 4,
         "group": 32, "g": 64, "per_channel": True, "update": True},
        # read-back of four sequences of one layer, a ragged token count
        {"name": "dequantize_ragged", "kind": "dequantize", "batch": 4, "heads": 8, "n": 8191, "dtype": "bf16",
         "bits": 4, "group": 128, "per_channel": False},
        # one layer of a decode step: 64 sequences of about two thousand tokens
        {"name": "scores_batch", "kind": "scores", "batch": 64, "heads": 8, "n": 2080, "qpk": 4, "dtype": "bf16",
         "bits": 2, "group": 32, "per_channel": False, "rope": False},
        # one layer of a decode step of a single long sequence, keys stored before the rotary embedding, per channel
        {"name": "scores_rope_single", "kind": "scores", "batch": 1, "heads": 8, "n": 32768, "qpk": 4, "dtype": "bf16",
         "bits": 2, "group": 32, "per_channel": True, "rope": True},
        # a short generation: prefill of an odd prompt, 40 decoded tokens (one or two flushes among them), values too
        {"name": "cache_generate", "kind": "cache", "batch": 8, "heads": 8, "qpk": 4, "n": 1003, "steps": 40,
         "dtype": "bf16", "bits": 2, "group": 32, "g": 32, "residual": 32, "values": True, "per_channel": False,
         "rope": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _setting(rng):
    """(r, lambda, g) around the paper's hyper-parameters."""
    return (rng.choice([5, 8, 10, 16, 20, 32, 40, 60, 64]), rng.choice([5e-4, 1e-3]), rng.choice([32, 64]))


def draw(rng):
    kind = rng.choice(["subspace", "prepare", "quantize", "quantize", "dequantize", "scores", "scores", "path", "cache"])
    r, lam, g = _setting(rng)
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    bits, group = rng.choice([2, 4]), rng.choice([32, 64, 128])
    pc = rng.random() < 0.4
    if kind == "subspace":
        heads, qpk = _log(rng, 1, 256), rng.choice([1, 2, 4, 8])
        n = min(_log(rng, 200, 32768), max(200, (1 << 23) // (heads * qpk)))
        return {"kind": kind, "heads": heads, "qpk": qpk, "n": n, "dtype": dtype, "r": r}
    if kind == "prepare":
        return {"kind": kind, "heads": _log(rng, 1, 256), "r": r, "lam": lam, "g": g, "full": rng.random() < 0.3}
    if kind == "path":
        heads, qpk = _log(rng, 1, 64), rng.choice([1, 2, 4, 8])
        n = min(_log(rng, 200, 16384), max(200, (1 << 22) // (heads * qpk)))
        keep = n % 32 if pc else rng.choice([0, 32, 128])
        return {"kind": kind, "heads": heads, "qpk": qpk, "n": n, "keep": keep, "dtype": dtype, "r": r, "lam": lam,
                "bits": bits, "group": 32 if pc else group, "g": g, "per_channel": pc}
    if kind == "cache":
        residual = rng.choice([32, 64, 128])
        return {"kind": kind, "batch": _log(rng, 1, 16), "heads": _log(rng, 1, 32), "qpk": rng.choice([1, 2, 4, 8]),
                "n": _log(rng, 20, 2000), "steps": rng.randint(8, 40), "dtype": rng.choice(["bf16", "f16"]),
                "bits": bits, "group": group, "g": g, "residual": residual, "values": rng.random() < 0.5,
                "per_channel": pc, "rope": rng.random() < 0.4}
    batch, heads = _log(rng, 1, 64), _log(rng, 1, 64)
    n = min(_log(rng, 32, 32768), max(32, (1 << 22) // (batch * heads)))
    if pc:
        n, group = n // 32 * 32, 32
    c = {"kind": kind, "batch": batch, "heads": heads, "n": n, "dtype": dtype, "bits": bits, "group": group,
         "per_channel": pc}
    if kind == "quantize":
        c.update(g=g, update=rng.random() < 0.85)
    if kind == "scores":
        c.update(qpk=rng.choice([1, 2, 4, 8]), rope=rng.random() < 0.4)
    return c


# ---- inputs ---------------------------------------------------------------------------------------------------- #

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)


def _directions(seed, heads):
    """Per head: 128 orthonormal directions (one random basis, in an order of the head's own) and their gains, which
    fall by 5 per cent from one to the next."""
    rng = np.random.Generator(np.random.PCG64(seed))
    basis, _ = np.linalg.qr(rng.standard_normal((D, D)))
    order = np.stack([rng.permutation(D) for _ in range(heads)])
    return torch.from_numpy(basis), order, 0.95 ** np.arange(D)


def _queries(seed, heads, qpk, n, dtype):
    """[heads*qpk, n, 128] on the GPU."""
    gen = _gen(seed)
    basis, order, gain = _directions(seed, heads)
    basis = basis.float().to(DEV)
    q = torch.empty((heads * qpk, n, D), dtype=dtype, device=DEV)
    per = max(1, (1 << 27) // (qpk * n * D))
    for h in range(0, heads, per):
        m = min(per, heads - h)
        x = _rand(gen, m, qpk * n, D)
        col = np.empty((m, D), dtype=np.float32)
        for j in range(m):
            col[j, order[h + j]] = gain
        x *= torch.from_numpy(col).to(DEV)[:, None, :]
        q[h * qpk:(h + m) * qpk] = (x.view(-1, D) @ basis.T).view(m * qpk, n, D).to(dtype)
    return q


def _qhat(seed, heads, r, rows=32768):
    """[heads, r, 128] double on the host: the top-r directions times singular values of `rows` pooled queries."""
    basis, order, gain = _directions(seed, heads)
    s = math.sqrt(rows) * torch.from_numpy(gain[:r])
    return torch.stack([basis[:, torch.from_numpy(o[:r])].T * s[:, None] for o in order])


def _keys(seed, batch, heads, n, dtype):
    """[batch, heads, n, 128] on the GPU, 2 to 6 outlier channels per head."""
    gen = _gen(seed + 7919)
    rng = np.random.Generator(np.random.PCG64(seed + 7919))
    fac = np.ones((heads, 1, D), dtype=np.float32)
    for h in range(heads):
        idx = rng.choice(D, size=int(rng.integers(2, 7)), replace=False)
        fac[h, 0, idx] = rng.uniform(8.0, 15.0, size=len(idx))
    fac = torch.from_numpy(fac).to(DEV)
    k = torch.empty((batch, heads, n, D), dtype=dtype, device=DEV)
    per = max(1, (1 << 27) // (max(1, n) * D))
    for b in range(batch):
        for h in range(0, heads, per):
            m = min(per, heads - h)
            k[b, h:h + m] = (_rand(gen, m, n, D) * fac[h:h + m]).to(dtype)
    return k


def _update(qhat, lam, g):
    """Lemma 2's panels in 64 bits from qhat [heads, r, 128] (double, host): U[tg:, (t-1)g:tg]."""
    heads, r, _ = qhat.shape
    u = torch.zeros((heads, D, D), dtype=torch.float64)
    eye = torch.eye(r, dtype=torch.float64) / lam
    for t in range(1, D // g):
        qb, qr = qhat[:, :, (t - 1) * g:t * g], qhat[:, :, t * g:]
        u[:, t * g:, (t - 1) * g:t * g] = -qr.transpose(1, 2) @ torch.linalg.solve(eye + qr @ qr.transpose(1, 2), qb)
    return u


def _stored_update(seed, heads, g):
    """An update matrix as a program holds it: r = 16, lambda = 1e-3, entries on the fp16 grid."""
    return _update(_qhat(seed + 104729, heads, 16), 1e-3, g).half().float().to(DEV)


def _pack_token(c, bits):
    """codes [..., n, 128] -> int32 words [..., n, 4 * bits]: channel c in word c // (32 / bits)."""
    per = 32 // bits
    w = c.to(torch.int64).view(*c.shape[:-1], D // per, per) << (bits * torch.arange(per, device=c.device))
    return _int32(w.sum(-1))


def _pack_channel(c, bits):
    """codes [..., n, 128] -> int32 words [..., n / 32, 128, bits]: token j of a group in word j // (32 / bits)."""
    per = 32 // bits
    t = c.to(torch.int64).view(*c.shape[:-2], -1, 32, D).transpose(-1, -2)
    w = t.reshape(*t.shape[:-1], bits, per) << (bits * torch.arange(per, device=c.device))
    return _int32(w.sum(-1))


def _int32(w):
    return torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)


def _round_to_nearest(x, lo, hi, bits):
    """(codes, scale, zero, dequantized) of x with the statistics (lo, hi), scale and zero in fp16."""
    scale = ((hi - lo) / ((1 << bits) - 1)).half()
    zero = lo.half()
    s, z = scale.to(x.dtype), zero.to(x.dtype)
    c = torch.round((x - z) / torch.where(s > 0, s, torch.ones_like(s))).clamp(0, (1 << bits) - 1)
    c = torch.where(s > 0, c, torch.zeros_like(c))
    return c, scale, zero, c * s + z


def _quantize(k, u, bits, group, g, per_channel):
    """Algorithm 1's Quant on k [..., n, 128] (its last two dimensions; u [..., 128, 128] or None) in k's own
    precision: (codes [..., n, 128], scale, zero, dequantized)."""
    x = k.clone()
    codes = torch.empty_like(x)
    ng = D // group if not per_channel else 0
    if per_channel:
        n = x.shape[-2]
        scale = torch.empty((*x.shape[:-2], n // 32, D), dtype=torch.float16, device=x.device)
    else:
        scale = torch.empty((*x.shape[:-1], ng), dtype=torch.float16, device=x.device)
    zero = torch.empty_like(scale)
    for t in range(D // g):
        b0, b1 = t * g, (t + 1) * g
        cur = x[..., b0:b1].clone()
        if per_channel:
            v = cur.view(*x.shape[:-2], n // 32, 32, g)
            c, s, z, y = _round_to_nearest(v, v.amin(-2, True), v.amax(-2, True), bits)
            scale[..., b0:b1], zero[..., b0:b1] = s.squeeze(-2), z.squeeze(-2)
            codes[..., b0:b1], x[..., b0:b1] = c.reshape(cur.shape), y.reshape(cur.shape)
        else:
            for j in range(b0 // group, max(b0 // group + 1, b1 // group)):
                if j * group >= b0:                       # a group's statistics are taken when it is reached
                    seg = x[..., j * group:(j + 1) * group]
                    lo, hi = seg.amin(-1), seg.amax(-1)
                    scale[..., j] = ((hi - lo) / ((1 << bits) - 1)).half()
                    zero[..., j] = lo.half()
                a, e = max(b0, j * group), min(b1, (j + 1) * group)
                s, z = scale[..., j:j + 1].to(x.dtype), zero[..., j:j + 1].to(x.dtype)
                c = torch.round((x[..., a:e] - z) / torch.where(s > 0, s, torch.ones_like(s)))
                c = torch.where(s > 0, c.clamp(0, (1 << bits) - 1), torch.zeros_like(c))
                codes[..., a:e], x[..., a:e] = c, c * s + z
        if u is not None and b1 < D:
            x[..., b1:] += (x[..., b0:b1] - cur) @ u[..., b1:, b0:b1].transpose(-1, -2).contiguous()
    return codes, scale, zero, x


def _in_chunks(k, u, bits, group, g, per_channel):
    """_quantize in 64 bits, a few heads at a time: (packed codes, scale, zero) as the library stores them."""
    pack = _pack_channel if per_channel else _pack_token
    out = []
    heads = k.shape[1]
    per = max(1, (1 << 19) // (k.shape[0] * max(1, k.shape[2])))
    for h in range(0, heads, per):
        c, s, z, _ = _quantize(k[:, h:h + per].double(), None if u is None else u[h:h + per].double(), bits, group, g,
                               per_channel)
        out.append((pack(c, bits), s, z))
    return tuple(torch.cat([o[i] for o in out], 1) for i in range(3))


def _store(seed, c):
    """A packed store, made in plain torch: keys quantized by plain round-to-nearest in fp32.
    (codes, scale, zero) as the library lays them out."""
    batch, heads, n, bits, group = c["batch"], c["heads"], c["n"], c["bits"], c["group"]
    pack = _pack_channel if c["per_channel"] else _pack_token
    k = _keys(seed, batch, heads, n, torch.float32)
    out = []
    for h in range(0, heads, 4):
        x, s, z, _ = _quantize(k[:, h:h + 4], None, bits, group, max(32, group), c["per_channel"])
        out.append((pack(x, bits), s, z))
    return tuple(torch.cat([o[i] for o in out], 1).contiguous() for i in range(3))


def _unpack(codes, bits, per_channel):
    """int32 words -> codes [..., n, 128] in 64 bits."""
    sh = bits * torch.arange(32 // bits, device=codes.device)
    c = ((codes.to(torch.int64)[..., None] >> sh) & ((1 << bits) - 1)).double()
    if not per_channel:
        return c.flatten(-2)
    return c.flatten(-2).transpose(-1, -2).flatten(-3, -2)


def _dequantized(codes, scale, zero, bits, group, per_channel):
    x = _unpack(codes, bits, per_channel)
    if per_channel:
        s, z = (v.double().repeat_interleave(32, -2) for v in (scale, zero))
    else:
        s, z = (v.double().repeat_interleave(group, -1) for v in (scale, zero))
    return x * s + z


def _inv_freq():
    return (10000.0 ** (-torch.arange(64, dtype=torch.float64) / 64.0)).float().to(DEV)


def _rotated(x, inv_freq, pos0):
    """Rotary embedding of x [..., n, 128] in 64 bits, token t at position pos0 + t."""
    a = (pos0 + torch.arange(x.shape[-2], device=x.device, dtype=torch.float64))[:, None] * inv_freq.double()
    c, s = torch.cos(a), torch.sin(a)
    lo, hi = x[..., :64], x[..., 64:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _logits(q, k, qpk, out_scale):
    """q [B, H*qpk, 128], k [B, H, n, 128] -> [B, H*qpk, n], in 64 bits."""
    b, h, n, _ = k.shape
    return (q.double().view(b, h, qpk, D) @ k.transpose(-1, -2).contiguous()).view(b, h * qpk, n) * out_scale


OUT_SCALE = 1.0 / math.sqrt(D)
POS0 = 5


def prepare(case, seed):
    c = dict(case)
    dt = DTYPES[c["dtype"]] if "dtype" in c else None
    kind = c["kind"]
    if kind == "subspace":
        return {"c": c, "q": _queries(seed, c["heads"], c["qpk"], c["n"], dt)}
    if kind == "prepare":
        return {"c": c, "qhat": _qhat(seed, c["heads"], c["r"]).float().to(DEV)}
    if kind == "quantize":
        return {"c": c, "k": _keys(seed, c["batch"], c["heads"], c["n"], dt),
                "u": _stored_update(seed, c["heads"], c["g"]) if c["update"] else None}
    if kind == "dequantize":
        return {"c": c, "store": _store(seed, c)}
    if kind == "scores":
        q = _rand(_gen(seed + 15485863), c["batch"], c["heads"] * c["qpk"], D).to(dt)
        return {"c": c, "store": _store(seed, c), "q": q, "inv_freq": _inv_freq()}
    if kind == "path":
        return {"c": c, "q": _queries(seed, c["heads"], c["qpk"], c["n"], dt), "k": _keys(seed, 1, c["heads"], c["n"], dt)}
    if kind == "cache":
        b, h, total = c["batch"], c["heads"], c["n"] + c["steps"]
        u = _stored_update(seed, h, c["g"])
        k = _keys(seed, b, h, total, dt)
        v = _rand(_gen(seed + 32452843), b, h, total, D).to(dt) if c["values"] else None
        q = _rand(_gen(seed + 15485863), c["steps"], b, h * c["qpk"], D).to(dt)
        m = -(-total // c["residual"]) * c["residual"]
        cache = squat.Cache(b, h, c["qpk"], c["bits"], c["group"], c["g"], c["residual"], m, dt, u, c["values"], DEV,
                            D, c["per_channel"])
        steps = range(c["n"], total)
        return {"c": c, "cache": cache, "k": k, "v": v, "q": q, "inv_freq": _inv_freq(),
                "kn": [k[:, :, t] for t in steps], "vn": [v[:, :, t] if v is not None else None for t in steps]}
    raise ValueError(kind)


def run(state):
    c = state["c"]
    kind = c["kind"]
    if kind == "subspace":
        qhat, eig, _ = squat.build_subspace(state["q"], c["qpk"], c["r"])
        return {"qhat": qhat, "eig": eig}
    if kind == "prepare":
        return {"update": squat.prepare(state["qhat"], c["lam"], c["g"], full_precision=c["full"])}
    if kind == "quantize":
        f = squat.quantize_keys_per_channel if c["per_channel"] else squat.quantize_keys
        codes, scale, zero = f(state["k"], state["u"], c["bits"], c["group"], c["g"])
        return {"codes": codes, "scale": scale, "zero": zero}
    if kind == "dequantize":
        f = squat.dequantize_keys_per_channel if c["per_channel"] else squat.dequantize_keys
        return {"k": f(*state["store"], c["bits"], c["group"], DTYPES[c["dtype"]])}
    if kind == "scores":
        codes, scale, zero = state["store"]
        if c["per_channel"]:
            if c["rope"]:
                s = squat.key_scores_rope_per_channel(state["q"], codes, scale, zero, c["bits"], c["qpk"],
                                                      state["inv_freq"], POS0, OUT_SCALE)
            else:
                s = squat.key_scores_per_channel(state["q"], codes, scale, zero, c["bits"], c["qpk"], OUT_SCALE)
        elif c["rope"]:
            s = squat.key_scores_rope(state["q"], codes, scale, zero, c["bits"], c["group"], c["qpk"],
                                      state["inv_freq"], POS0, OUT_SCALE)
        else:
            s = squat.key_scores(state["q"], codes, scale, zero, c["bits"], c["group"], c["qpk"], OUT_SCALE)
        return {"scores": s}
    if kind == "path":
        qhat, eig, _ = squat.build_subspace(state["q"], c["qpk"], c["r"])
        u = squat.prepare(qhat, c["lam"], c["g"])
        k = state["k"][:, :, :c["n"] - c["keep"]]
        if c["per_channel"]:
            codes, scale, zero = squat.quantize_keys_per_channel(k, u, c["bits"], c["group"], c["g"])
        else:
            codes, scale, zero = squat.quantize_keys(k, u, c["bits"], c["group"], c["g"])
        return {"qhat": qhat, "eig": eig, "update": u, "codes": codes, "scale": scale, "zero": zero}
    if kind == "cache":
        cache = state["cache"]
        cache.reset()
        cache.prefill(state["k"][:, :, :c["n"]], state["v"][:, :, :c["n"]] if c["values"] else None)
        logits = []
        for t in range(c["steps"]):
            cache.append(state["kn"][t], state["vn"][t])
            if c["rope"]:
                logits.append(cache.key_scores_rope(state["q"][t], state["inv_freq"], POS0, OUT_SCALE))
            else:
                logits.append(cache.key_scores(state["q"][t], OUT_SCALE))
        out = {"logits": logits}
        cnt, st = cache.counts(), cache.stores()
        rows = cnt.keys_quantized // 32 if c["per_channel"] else cnt.keys_quantized
        for name in ("codes", "scale", "zero"):
            out["key_" + name] = st["key_" + name][:, :, :rows]
            if c["values"]:
                out["value_" + name] = st["value_" + name][:, :, :cnt.values_quantized]
        return out
    raise ValueError(kind)


# ---- what a pass cannot do without ------------------------------------------------------------------------------ #

def _store_bytes(keys, bits, group, per_channel):
    return keys * (D * bits / 8 + (4 * D / 32 if per_channel else 4 * D / group))


def _solve_flops(heads, r):
    """Tridiagonal reduction of a 128 x 128 matrix and r vectors carried back through it."""
    return heads * (4.0 / 3.0 * D ** 3 + 2.0 * r * D ** 2)


def _panel_flops(heads, r, g):
    """Per panel: Qr Qr^T (half of it), a factorisation, two solves for g columns, the product with Qr^T."""
    return heads * sum(r * r * m + r ** 3 / 3 + 2 * r * r * g + 2 * m * r * g for m in range(D - g, 0, -g))


def _update_flops(g):
    return sum(2 * g * m for m in range(D - g, 0, -g))


def work(case):
    c = case
    size = {"bf16": 2, "f16": 2, "f32": 4}.get(c.get("dtype"), 0)
    kind, h = c["kind"], c["heads"]
    if kind == "subspace":
        rows = h * c["qpk"] * c["n"]
        return {"bytes": rows * D * size + h * c["r"] * (D + 1) * 4,
                "flops": 2.0 * D * D * rows + _solve_flops(h, c["r"])}
    if kind == "prepare":
        return {"bytes": h * D * (c["r"] + D) * 4, "flops": _panel_flops(h, c["r"], c["g"])}
    if kind == "path":
        rows, keys = h * c["qpk"] * c["n"], h * (c["n"] - c["keep"])
        return {"bytes": rows * D * size + h * (c["r"] * (D + 1) + D * D) * 4 + keys * D * size +
                _store_bytes(keys, c["bits"], c["group"], c["per_channel"]),
                "flops": 2.0 * D * D * rows + _solve_flops(h, c["r"]) + _panel_flops(h, c["r"], c["g"]) +
                keys * _update_flops(c["g"])}
    if kind == "cache":
        b, steps = c["batch"] * h, c["steps"]
        nbytes = b * (c["n"] + steps) * D * size * (2 if c["values"] else 1) + b * steps * c["qpk"] * D * size
        nbytes += _store_bytes(b * (c["n"] + steps), c["bits"], c["group"], c["per_channel"])
        for t in range(1, steps + 1):
            total = c["n"] + t
            old = total // c["residual"] * c["residual"]
            nbytes += _store_bytes(b * old, c["bits"], c["group"], c["per_channel"]) + b * (total - old) * D * size
            nbytes += b * c["qpk"] * total * 4
        return {"bytes": nbytes, "flops": b * (c["n"] + steps) * _update_flops(c["g"]) +
                b * steps * 2.0 * D * c["qpk"] * (c["n"] + steps / 2)}
    keys = c["batch"] * h * c["n"]
    packed = _store_bytes(keys, c["bits"], c["group"], c["per_channel"])
    if kind == "quantize":
        return {"bytes": keys * D * size + packed + (h * D * D * 4 if c["update"] else 0),
                "flops": keys * (8.0 * D + (_update_flops(c["g"]) if c["update"] else 0))}
    if kind == "dequantize":
        return {"bytes": packed + keys * D * size, "flops": 2.0 * D * keys}
    return {"bytes": packed + c["batch"] * h * c["qpk"] * D * size + keys * c["qpk"] * 4,
            "flops": 2.0 * D * keys * c["qpk"]}


def tolerance(case):
    """About four times the distance of the outputs from `exact`, over 200 drawn cases (largest seen in brackets)."""
    c = case
    kind = c["kind"]
    if kind == "subspace":                                # fp32 sums of the Gram matrix (1.1e-6, 1.7e-5)
        return {"rel": 5e-6, "max": 8e-5}
    if kind == "prepare":                                 # stored in fp32 (3.2e-8) or on the fp16 grid (2.1e-4, 4.9e-4)
        return {"rel": 2e-7, "max": 1e-6} if c["full"] else {"rel": 8e-4, "max": 2e-3}
    if kind == "dequantize":                              # one rounding to the output type (bf16: 1.7e-3, 3.9e-3)
        return {"bf16": {"rel": 4e-3, "max": 8e-3}, "f16": {"rel": 5e-4, "max": 1e-3},
                "f32": {"rel": 2e-7, "max": 1e-6}}[c["dtype"]]
    if kind == "scores":                                  # rotated in fp16 (3.2e-4, 3.4e-3), plain (6e-7, 6.3e-6)
        return {"rel": 1.3e-3, "max": 1.4e-2} if c["rope"] else {"rel": 3e-6, "max": 3e-5}
    # A value on a rounding boundary may fall to either side; what follows it in the same key then differs too
    # (words of codes 5.9e-3, scales and zero-points 1.7e-3; a single one by more than half its size)
    if kind == "cache":                                   # logits against such keys: 3.7e-2
        return {"rel": 3e-2, "max": 0.99, "differ": 1e-2}
    return {"rel": 7e-3, "max": 0.99, "differ": 1e-2}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------- #

def _top_directions(q, qpk, r):
    """(qhat, eig) in 64 bits of q [heads*qpk, n, 128]; every row's largest component is positive."""
    heads = q.shape[0] // qpk
    q = q.view(heads, -1, D)
    gram = torch.zeros((heads, D, D), dtype=torch.float64, device=q.device)
    for h in range(heads):
        for t in range(0, q.shape[1], 1 << 18):
            x = q[h, t:t + (1 << 18)].double()
            gram[h] += x.T @ x
    eig, vec = torch.linalg.eigh(gram.cpu())
    eig, vec = eig.flip(-1)[:, :r].clamp_min(0), vec.flip(-1)[:, :, :r].transpose(1, 2)
    big = vec.gather(-1, vec.abs().argmax(-1, keepdim=True))
    return (vec * torch.sign(big) * eig.sqrt()[..., None]).contiguous(), eig


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "cache":
        return _exact_cache(c, seed)
    s = prepare(c, seed)
    if kind == "subspace":
        qhat, eig = _top_directions(s["q"], c["qpk"], c["r"])
        return {"qhat": qhat, "eig": eig}
    if kind == "prepare":
        return {"update": _update(s["qhat"].cpu().double(), c["lam"], c["g"])}
    if kind == "quantize":
        codes, scale, zero = _in_chunks(s["k"], s["u"], c["bits"], c["group"], c["g"], c["per_channel"])
        return {"codes": codes, "scale": scale.double(), "zero": zero.double()}
    if kind == "dequantize":
        return {"k": _dequantized(*s["store"], c["bits"], c["group"], c["per_channel"])}
    if kind == "scores":
        out = []
        for b in range(c["batch"]):
            k = _dequantized(*(x[b:b + 1] for x in s["store"]), c["bits"], c["group"], c["per_channel"])
            if c["rope"]:
                k = _rotated(k, s["inv_freq"], POS0)
            out.append(_logits(s["q"][b:b + 1], k, c["qpk"], OUT_SCALE))
        return {"scores": torch.cat(out)}
    qhat, eig = _top_directions(s["q"], c["qpk"], c["r"])
    u = _update(qhat, c["lam"], c["g"])
    k = s["k"][:, :, :c["n"] - c["keep"]]
    codes, scale, zero = _in_chunks(k, u.half().to(DEV), c["bits"], c["group"], c["g"], c["per_channel"])
    return {"qhat": qhat, "eig": eig, "update": u, "codes": codes, "scale": scale.double(), "zero": zero.double()}


def _exact_cache(c, seed):
    """What is quantized does not depend on when it was: a key's codes depend on the key alone (per channel: on its
    aligned group of 32 tokens)."""
    s = prepare(c, seed)
    total = c["n"] + c["steps"]
    old = total // c["residual"] * c["residual"]
    out = {"logits": []}
    codes, scale, zero = _in_chunks(s["k"][:, :, :old], s["cache"].update, c["bits"], c["group"], c["g"],
                                    c["per_channel"])
    deq = _dequantized(codes, scale, zero, c["bits"], c["group"], c["per_channel"])
    full = s["k"].double()
    if c["rope"]:
        deq, full = _rotated(deq, s["inv_freq"], POS0), _rotated(full, s["inv_freq"], POS0)
    for t in range(c["steps"]):
        now = c["n"] + t + 1
        cut = now // c["residual"] * c["residual"]
        out["logits"].append(_logits(s["q"][t], torch.cat([deq[:, :, :cut], full[:, :, cut:now]], 2), c["qpk"],
                                     OUT_SCALE))
    out.update(key_codes=codes, key_scale=scale.double(), key_zero=zero.double())
    if c["values"]:
        v = s["v"][:, :, :max(0, total - c["residual"])]
        codes, scale, zero = _in_chunks(v, None, c["bits"], c["group"], max(32, c["group"]), False)
        out.update(value_codes=codes, value_scale=scale.double(), value_zero=zero.double())
    return out
