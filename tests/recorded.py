"""Runs the library's host side against a stand-in for the HIP runtime's launch calls (launch_recorder.c): the process that
calls `start` must not have loaded the real runtime into its global scope, so tests run a child for it (`run`)."""
import ctypes
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class Launch(ctypes.Structure):
    _fields_ = [("func", ctypes.c_uint64), ("grid", ctypes.c_uint32 * 3), ("block", ctypes.c_uint32 * 3),
                ("head", ctypes.c_uint64 * 2), ("failed", ctypes.c_int), ("shared", ctypes.c_uint64)]


class CacheConfig(ctypes.Structure):
    _fields_ = [("n_batch", ctypes.c_int64), ("n_kv_heads", ctypes.c_int), ("q_per_kv", ctypes.c_int),
                ("d", ctypes.c_int), ("bits", ctypes.c_int), ("group", ctypes.c_int), ("g", ctypes.c_int),
                ("residual", ctypes.c_int), ("max_tokens", ctypes.c_int64), ("kv_dtype", ctypes.c_int),
                ("quantize_values", ctypes.c_int), ("key_per_channel", ctypes.c_int)]


class CacheCounts(ctypes.Structure):
    _fields_ = [("n_tokens", ctypes.c_int64), ("keys_quantized", ctypes.c_int64), ("keys_residual", ctypes.c_int),
                ("values_quantized", ctypes.c_int64), ("values_residual", ctypes.c_int), ("value_ring_head", ctypes.c_int)]


def run(recorder: str, code: str):
    """Runs `code` (which prints one JSON line) in a child that has neither torch nor the real runtime loaded."""
    prog = "import sys, ctypes, json; sys.path.insert(0, %r); import recorded as R; rec, lib = R.start(%r)\n%s" % (HERE, recorder, code)
    p = subprocess.run([sys.executable, "-c", prog], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stderr
    return json.loads(p.stdout.strip().splitlines()[-1])


def build(folder: str) -> str:
    so = os.path.join(folder, "launch_recorder.so")
    subprocess.run(["cc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "launch_recorder.c"), "-o", so], check=True)
    return so


def start(recorder: str):
    rec = ctypes.CDLL(recorder, ctypes.RTLD_GLOBAL)
    rec.launch_at.restype = ctypes.POINTER(Launch)
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2503_24358_amd", "libsquat.so"))
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    lib.squat_cache_arena_bytes.restype = ctypes.c_size_t
    lib.squat_cache_create.argtypes = [vp, vp, ctypes.c_size_t, vp, vp]
    lib.squat_cache_state.argtypes = [vp, vp]
    lib.squat_cache_prefill.argtypes = [vp, vp, vp, i64, i64, i64, i64, vp]
    lib.squat_cache_append.argtypes = [vp, vp, vp, i64, i64, vp]
    lib.squat_cache_key_scores.argtypes = [vp, vp, ctypes.c_int, i64, i64, ctypes.c_float, vp, i64, i64, vp]
    lib.squat_build_subspace_workspace.restype = ctypes.c_size_t
    lib.squat_build_subspace_workspace.argtypes = [i64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    lib.squat_build_subspace.argtypes = [vp, ctypes.c_int, i64, ctypes.c_int, ctypes.c_int, ctypes.c_int, i64, i64, ctypes.c_int,
                                         vp, vp, vp, vp, ctypes.c_size_t, vp]
    lib.squat_key_scores.argtypes = [vp, vp, vp, i64, ctypes.c_int, i64, ctypes.c_int, ctypes.c_int, ctypes.c_int, vp, ctypes.c_int,
                                     ctypes.c_int, i64, i64, ctypes.c_float, vp, i64, i64, vp]
    return rec, lib


def cache(lib, **kw):
    """A cache on made-up device addresses (nothing runs, nothing is read)."""
    c = dict(n_batch=1, n_kv_heads=3, q_per_kv=1, d=128, bits=2, group=32, g=32, residual=4, max_tokens=64, kv_dtype=2,
             quantize_values=1, key_per_channel=0)
    c.update(kw)
    cfg = CacheConfig(*[c[n] for n, _ in CacheConfig._fields_])
    h = ctypes.c_void_p()
    n = lib.squat_cache_arena_bytes(ctypes.byref(cfg))
    assert n > 0
    assert lib.squat_cache_create(ctypes.byref(cfg), 0x100000, n, None, ctypes.byref(h)) == 0
    return h


def counts(lib, h):
    c = CacheCounts()
    assert lib.squat_cache_state(h, ctypes.byref(c)) == 0
    return [getattr(c, n) for n, _ in CacheCounts._fields_]
