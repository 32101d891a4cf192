"""The native part of the Python binding: what it refuses and with which exception, and that results land where the caller
says (given outputs, a stream's handle or object)."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2503_24358_amd import squat


def test_refuses_without_a_device():
    k = torch.zeros(1, 2, 32, 128)
    with pytest.raises(ValueError):
        squat.quantize_keys(k, None, 2, 32, 32)
    with pytest.raises(ValueError):
        squat.quantize_keys_per_channel(k, None, 2, 32, 32)
    codes, meta = torch.zeros(1, 2, 32, 8, dtype=torch.int32), torch.zeros(1, 2, 32, 4, dtype=torch.float16)
    with pytest.raises(ValueError):
        squat.dequantize_keys(codes, meta, meta, 2, 32)
    with pytest.raises(ValueError):
        squat.key_scores(torch.zeros(1, 2, 128), codes, meta, meta, 2, 32, 1)
    with pytest.raises(AttributeError):
        squat.quantize_keys("no tensor", None, 2, 32, 32)
    with pytest.raises(TypeError):
        squat.native().quantize_keys(k, None, 2, 32, 32)
    with pytest.raises(TypeError):
        squat.native().dequantize_keys(codes, meta, meta, 2, 32, torch.float32, None)


def _stores(device="cpu"):
    """(q, per-token store, per-channel store) of one sequence, two heads, 32 tokens."""
    q = torch.zeros(1, 2, 128, device=device)
    per_token = (torch.zeros(1, 2, 32, 8, dtype=torch.int32, device=device),
                 *(torch.zeros(1, 2, 32, 4, dtype=torch.float16, device=device) for _ in range(2)))
    per_channel = (torch.zeros(1, 2, 1, 128, 2, dtype=torch.int32, device=device),
                   *(torch.zeros(1, 2, 1, 128, dtype=torch.float16, device=device) for _ in range(2)))
    return q, per_token, per_channel


def test_logits_refuse_host_stores():
    """(The store a call reads; a host `out` beside device inputs is refused on the device, below.)"""
    q, per_token, per_channel = _stores()
    inv = torch.ones(64)
    with pytest.raises(ValueError):
        squat.key_scores_per_channel(q, *per_channel, 2, 1)
    with pytest.raises(ValueError):
        squat.key_scores_rope(q, *per_token, 2, 32, 1, inv)
    with pytest.raises(ValueError):
        squat.key_scores_rope_per_channel(q, *per_channel, 2, 1, inv)


def _host_or_pinned(t, pinned):
    return torch.empty(t.shape, dtype=t.dtype, pin_memory=pinned)


@pytest.mark.gpu
def test_host_memory_is_refused_pinned_memory_taken():
    """No launch sees a host pointer it cannot reach: every output, workspace and part of a store that used to go unchecked."""
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    k = torch.randn(1, 2, 32, 128, generator=g, device="cuda")
    q = torch.randn(1, 2, 128, generator=g, device="cuda")
    inv = torch.ones(64, device="cuda")
    per_token, per_channel = squat.quantize_keys(k, None, 2, 32, 32), squat.quantize_keys_per_channel(k, None, 2, 32, 32)
    cache = squat.Cache(1, 2, 1, 2, 32, 32, 32, 64, torch.float32)
    cache.append(q)
    qhat = torch.randn(2, 4, 128, generator=g, device="cuda")
    names = ("codes", "scale", "zero")
    calls = [(lambda i=i, f=f, **kw: f(k, None, 2, 32, 32, **kw)[i], n) for f in (squat.quantize_keys, squat.quantize_keys_per_channel)
             for i, n in enumerate(names)]
    calls += [(lambda **kw: squat.dequantize_keys(*per_token, 2, 32, torch.float32, **kw), "out"),
              (lambda **kw: squat.dequantize_keys_per_channel(*per_channel, 2, 32, torch.float32, **kw), "out"),
              (lambda **kw: squat.key_scores(q, *per_token, 2, 32, 1, **kw), "out"),
              (lambda **kw: squat.key_scores_rope(q, *per_token, 2, 32, 1, inv, **kw), "out"),
              (lambda **kw: squat.key_scores_per_channel(q, *per_channel, 2, 1, **kw), "out"),
              (lambda **kw: squat.key_scores_rope_per_channel(q, *per_channel, 2, 1, inv, **kw), "out"),
              (lambda **kw: cache.key_scores(q, **kw), "out"),
              (lambda **kw: cache.key_scores_rope(q, inv, **kw), "out"),
              (lambda **kw: squat.build_subspace(q.view(2, 1, 128), 1, 1, **kw)[0], "qhat"),
              (lambda **kw: squat.prepare(qhat, 1e-3, 32, **kw), "update")]
    for call, name in calls:
        want = call()
        with pytest.raises(ValueError):
            call(**{name: _host_or_pinned(want, False)})
        got = call(**{name: _host_or_pinned(want, True)})
        torch.cuda.synchronize()
        assert not got.is_cuda and torch.equal(got, want.cpu())
    for i in range(3):
        for logits, store in ((lambda *s: squat.key_scores_rope(q, *s, 2, 32, 1, inv), per_token),
                              (lambda *s: squat.key_scores_per_channel(q, *s, 2, 1), per_channel),
                              (lambda *s: squat.key_scores_rope_per_channel(q, *s, 2, 1, inv), per_channel)):
            with pytest.raises(ValueError):
                logits(*[t.cpu() if j == i else t for j, t in enumerate(store)])
    with pytest.raises(ValueError):
        squat.key_scores_per_channel(q.cpu(), *per_channel, 2, 1)
    want, pinned = squat.key_scores_per_channel(q, *per_channel, 2, 1), [t.cpu().pin_memory() for t in per_channel]
    with pytest.raises(ValueError):                    # (where would the logits lie?)
        squat.key_scores_per_channel(q, *pinned, 2, 1)
    assert torch.equal(squat.key_scores_per_channel(q, *pinned, 2, 1, out=torch.empty_like(want)), want)
    with pytest.raises(ValueError):
        squat.prepare(qhat, 1e-3, 32, ws=torch.empty(1 << 20, dtype=torch.uint8))
    with pytest.raises(ValueError):
        squat.Cache(1, 2, 1, 2, 32, 32, 32, 64, torch.float32, update=torch.zeros(2, 128, 128))


def test_rotary_logits_need_their_frequencies():
    q, per_token, per_channel = _stores()
    with pytest.raises(AttributeError):
        squat.key_scores_rope(q, *per_token, 2, 32, 1, None)
    with pytest.raises(AttributeError):
        squat.key_scores_rope_per_channel(q, *per_channel, 2, 1, None)


INTS = (np.int64, np.int32, np.uint8, torch.tensor)


@pytest.mark.parametrize("kind", INTS)
def test_what_stands_for_an_int_is_taken(kind):
    """(Taken: the next check, for a device tensor, is the one that refuses.)"""
    q, per_token, per_channel = _stores()
    bits, group, qpk = kind(2), kind(32), kind(1)
    inv = torch.ones(64)
    for call in (lambda b: squat.key_scores(q, *per_token, b, group, qpk), lambda b: squat.key_scores_per_channel(q, *per_channel, b, qpk),
                 lambda b: squat.key_scores_rope(q, *per_token, b, group, qpk, inv),
                 lambda b: squat.key_scores_rope_per_channel(q, *per_channel, b, qpk, inv)):
        with pytest.raises(ValueError):
            call(bits)
        with pytest.raises(TypeError):
            call(2.0)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", INTS)
def test_what_stands_for_an_int_gives_the_same(kind):
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    k = torch.randn(1, 2, 32, 128, generator=g, device="cuda")
    q = torch.randn(1, 2, 128, generator=g, device="cuda")
    inv = torch.rand(64, generator=g, device="cuda")

    def every_call(n):
        a = squat.quantize_keys(k, None, n(2), n(32), n(32))
        b = squat.quantize_keys_per_channel(k, None, n(2), n(32), n(32))
        return (*a, *b, squat.dequantize_keys(*a, n(2), n(32)), squat.dequantize_keys_per_channel(*b, n(2), n(32)),
                squat.key_scores(q, *a, n(2), n(32), n(1)), squat.key_scores_per_channel(q, *b, n(2), n(1)),
                squat.key_scores_rope(q, *a, n(2), n(32), n(1), inv, n(3)),
                squat.key_scores_rope_per_channel(q, *b, n(2), n(1), inv, n(3)))
    assert all(torch.equal(x, y) for x, y in zip(every_call(kind), every_call(int)))


@pytest.mark.gpu
def test_rotary_logits_need_their_frequencies_on_the_device():
    q, per_token, per_channel = _stores("cuda")
    with pytest.raises(AttributeError):
        squat.key_scores_rope(q, *per_token, 2, 32, 1, None)
    with pytest.raises(AttributeError):
        squat.key_scores_rope_per_channel(q, *per_channel, 2, 1, None)
    cache = squat.Cache(1, 2, 1, 2, 32, 32, 32, 64, torch.float32)
    cache.append(q)
    with pytest.raises(AttributeError):
        cache.key_scores_rope(q, None)


@pytest.mark.gpu
def test_refusals_on_the_device():
    k = torch.randn(1, 2, 32, 128, device="cuda")
    with pytest.raises(KeyError):
        squat.quantize_keys(k.double(), None, 2, 32, 32)
    with pytest.raises(ValueError):
        squat.quantize_keys(k[0], None, 2, 32, 32)
    with pytest.raises(ValueError):
        squat.quantize_keys(k, torch.zeros(2, 128, 128, device="cuda", dtype=torch.float64), 2, 32, 32)
    with pytest.raises(TypeError):
        squat.quantize_keys(k, None, 2.0, 32, 32)
    with pytest.raises(squat.SquatError) as e:
        squat.quantize_keys(k, None, 4, 16, 32)
    assert e.value.status < 0 and "squat_quantize_keys" in str(e.value)
    codes, scale, zero = squat.quantize_keys(k, None, 2, 32, 32)
    with pytest.raises(ValueError):
        squat.key_scores(k[:, :, 0, :64], codes, scale, zero, 2, 32, 1)
    with pytest.raises(ValueError):
        squat.key_scores(k[:, :, 0], codes[:, :, ::2], scale, zero, 2, 32, 1)
    with pytest.raises(ZeroDivisionError):
        squat.key_scores(k[:, :, 0], codes, scale, zero, 0, 32, 1)
    cache = squat.Cache(1, 2, 1, 2, 32, 32, 32, 64, torch.float32)
    with pytest.raises(squat.SquatError):
        cache.key_scores(k[:, :, 0, 1:])               # misaligned
    cache.append(k[:, :, 0])
    with pytest.raises(ValueError):
        cache.append(k[:, :, 0], k[:, :, 0].clone())    # other strides


@pytest.mark.gpu
def test_output_type_left_to_torch():
    k = torch.randn(1, 2, 32, 128, device="cuda")
    per_token, per_channel = squat.quantize_keys(k, None, 2, 32, 32), squat.quantize_keys_per_channel(k, None, 2, 32, 32)
    for call in (lambda t: squat.dequantize_keys(*per_token, 2, 32, t), lambda t: squat.dequantize_keys_per_channel(*per_channel, 2, 32, t)):
        assert torch.equal(call(None), call(torch.float32))
        with pytest.raises(TypeError):
            call("float32")
        with pytest.raises(KeyError):
            call(torch.float64)


@pytest.mark.gpu
def test_logits_into_more_dimensions():
    """The first three count: rows of tokens with a dimension of one behind them are a place like any other."""
    k = torch.randn(2, 2, 32, 128, device="cuda")
    q = torch.randn(2, 2, 128, device="cuda")
    inv = torch.ones(64, device="cuda")
    per_token, per_channel = squat.quantize_keys(k, None, 2, 32, 32), squat.quantize_keys_per_channel(k, None, 2, 32, 32)
    for call in (lambda **kw: squat.key_scores(q, *per_token, 2, 32, 1, **kw), lambda **kw: squat.key_scores_per_channel(q, *per_channel, 2, 1, **kw),
                 lambda **kw: squat.key_scores_rope(q, *per_token, 2, 32, 1, inv, **kw),
                 lambda **kw: squat.key_scores_rope_per_channel(q, *per_channel, 2, 1, inv, **kw)):
        out = torch.empty(2, 2, 32, 1, device="cuda")
        assert call(out=out) is out and torch.equal(out[..., 0], call())
        with pytest.raises(IndexError):
            call(out=torch.empty(4, 32, device="cuda"))


@pytest.mark.gpu
@pytest.mark.parametrize("half", ["0.5", np.float32(0.5), torch.tensor(0.5), np.array(0.5)])
def test_scale_is_what_float_takes(half):
    k = torch.randn(2, 2, 32, 128, device="cuda")
    q = torch.randn(2, 2, 128, device="cuda")
    store = squat.quantize_keys(k, None, 2, 32, 32)
    cache = squat.Cache(2, 2, 1, 2, 32, 32, 32, 64, torch.float32)
    cache.append(k[:, :, 0])
    for call in (lambda s: squat.key_scores(q, *store, 2, 32, 1, s), lambda s: cache.key_scores(q, s)):
        assert torch.equal(call(half), call(0.5))
        with pytest.raises(ValueError):
            call("half")
        with pytest.raises(TypeError):
            call(None)


@pytest.mark.gpu
def test_a_group_of_none():
    k = torch.randn(1, 2, 32, 128, device="cuda")
    codes, scale, zero = squat.quantize_keys(k, None, 2, 32, 32)
    with pytest.raises(ZeroDivisionError):               # (no shape for the outputs)
        squat.quantize_keys(k, None, 2, 0, 32)
    with pytest.raises(squat.SquatError):                # the library's answer
        squat.quantize_keys(k, None, 2, 0, 32, codes=codes, scale=scale, zero=zero)


@pytest.mark.gpu
def test_a_destroyed_cache():
    q = torch.randn(1, 2, 128, device="cuda")
    cache = squat.Cache(1, 2, 1, 2, 32, 32, 32, 64, torch.float32)
    cache.append(q)
    cache.__del__()
    for call in (lambda: cache.append(q), lambda: cache.key_scores(q), lambda: cache.key_scores_rope(q, torch.ones(64, device="cuda"))):
        with pytest.raises(squat.SquatError):
            call()


ALLOCATOR = """
extern int PyGILState_Check(void);
static void* block;
static int asked, held;
void lend(void* p) { block = p; }
int times_asked(void) { return asked; }
int times_held(void) { return held; }
void* get(long size, int device, void* stream) { ++asked; held += PyGILState_Check(); return block; }
void put(void* p, long size, int device, void* stream) {}
"""


# Lent: the memory 2 MiB into a tensor, an address that torch's own table of blocks does not hold.
ALLOCATING = """
import ctypes, os, sys, torch
sys.path.insert(0, sys.argv[2])
from paper_2503_24358_amd import squat
lib = ctypes.CDLL(sys.argv[1])
block = torch.zeros(66 << 20, dtype=torch.uint8, device="cuda")
lib.lend(ctypes.c_void_p(block.data_ptr() + (2 << 20)))
allocator = torch.cuda.memory.CUDAPluggableAllocator(sys.argv[1], "get", "put")
k = torch.randn(1, 2, 32, 128, device="cuda")
want = squat.quantize_keys(k, None, 2, 32, 32)
pool = torch.cuda.MemPool(allocator.allocator())
with torch.cuda.use_mem_pool(pool):
    got = squat.quantize_keys(k, None, 2, 32, 32)
torch.cuda.synchronize()
lent = all(block.data_ptr() <= t.data_ptr() < block.data_ptr() + block.numel() for t in got)
print(lib.times_asked(), lib.times_held(), lent, all(torch.equal(a, b) for a, b in zip(got, want)), flush=True)
os._exit(0)                                              # (lent memory is nothing for torch to clean up)
"""


@pytest.mark.gpu
def test_outputs_are_allocated_with_the_interpreter_free(tmp_path):
    """torch's allocator grows through a function that looks whether the calling thread holds the interpreter."""
    (tmp_path / "allocator.c").write_text(ALLOCATOR)
    so = str(tmp_path / "allocator.so")
    subprocess.run(["cc", "-O1", "-shared", "-fPIC", str(tmp_path / "allocator.c"), "-o", so], check=True)
    root = os.path.dirname(os.path.dirname(squat.__file__))
    p = subprocess.run([sys.executable, "-c", ALLOCATING, so, root], capture_output=True, text=True, timeout=100)
    assert p.returncode == 0, p.stderr
    assert p.stdout.split() == ["1", "0", "True", "True"]


@pytest.mark.gpu
def test_results_land_where_they_are_asked_for():
    k = torch.randn(2, 3, 40, 128, device="cuda", dtype=torch.float16)
    q = torch.randn(2, 6, 128, device="cuda", dtype=torch.bfloat16)
    want = squat.quantize_keys(k, None, 4, 64, 64)
    given = tuple(torch.empty_like(t) for t in want)
    got = squat.quantize_keys(k, None, 4, 64, 64, codes=given[0], scale=given[1], zero=given[2])
    assert all(a is b and torch.equal(b, w) for a, b, w in zip(got, given, want))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for stream in (side, side.cuda_stream):
        out = torch.zeros(2, 6, 50, device="cuda")
        side.wait_stream(torch.cuda.current_stream())
        assert squat.key_scores(q, *want, 4, 64, 2, 0.5, out=out, stream=stream) is out
        side.synchronize()
        assert torch.equal(out[:, :, :40], squat.key_scores(q, *want, 4, 64, 2, 0.5)) and not out[:, :, 40:].any()
    back = torch.empty(2, 3, 40, 128, device="cuda")
    assert squat.dequantize_keys(*want, 4, 64, out=back) is back
    assert torch.equal(back, squat.dequantize_keys(*want, 4, 64, torch.float32))
    with torch.cuda.stream(side):
        again = squat.dequantize_keys(*want, 4, 64, torch.float32)
    side.synchronize()
    assert torch.equal(again, back)
