"""Launches of squat_cache_key_scores for caches of many heads.  A grid's y and z hold 65535 each, so packed keys of head
counts without a divisor that suits are refused; full-precision keys alone are not bound by that.  Beside packed keys up to
24 MiB of them (in whole eights per head) are taken into the packed keys' launch.  Host side only, against a recorder of
the launches."""
import pytest

from . import recorded


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return recorded.build(str(tmp_path_factory.mktemp("recorder")))


CODE = """
h = R.cache(lib, n_batch=%(b)d, n_kv_heads=%(h)d, residual=%(r)d, max_tokens=%(r)d * 4, quantize_values=0, key_per_channel=%(pc)d, kv_dtype=%(dt)d)
assert lib.squat_cache_prefill(h, 0x10000, None, %(n)d, %(h)d * %(n)d * 128, %(n)d * 128, 128, None) == 0
n0 = rec.recorded()
rc = lib.squat_cache_key_scores(h, 0x10000, 2, %(h)d * 128, 128, 1.0, 0x20000, %(h)d * %(n)d, %(n)d, None)
print(json.dumps(dict(rc=rc, grids=[list(rec.launch_at(i).contents.grid) for i in range(n0, rec.recorded())])))
"""


@pytest.mark.parametrize("pc", [0, 1])
@pytest.mark.parametrize("b,h,n", [(1, 3, 2), (1, 65537, 2), (1, 131074, 31), (65537, 3, 31), (7, 65521, 1)])
def test_full_precision_keys_alone(recorder, b, h, n, pc):
    r = recorded.run(recorder, CODE % dict(b=b, h=h, n=n, r=32, pc=pc, dt=2))
    assert r["rc"] == 0 and len(r["grids"]) == 1
    x, y, z = r["grids"][0]
    assert y <= 65535 and z <= 65535 and x * y * z * 256 >= b * h * n * 8      # eight lanes per key


@pytest.mark.parametrize("pc", [0, 1])
def test_packed_keys_of_such_head_counts_stay_refused(recorder, pc):
    r = recorded.run(recorder, CODE % dict(b=1, h=65537, n=33, r=32, pc=pc, dt=2))
    assert r["rc"] == -2 and r["grids"] == []


@pytest.mark.parametrize("pc", [0, 1])
@pytest.mark.parametrize("b,h,n,r,dt,launches",
                         [(1, 3, 32, 32, 2, 1), (1, 3, 33, 32, 2, 1), (8, 1536, 40, 32, 2, 1), (8, 1536, 41, 32, 1, 2),
                          (1, 12289, 33, 32, 2, 2), (1, 6144, 40, 32, 0, 1), (1, 6145, 40, 32, 0, 2), (96, 1, 2047, 1024, 2, 1),
                          (97, 1, 2047, 1024, 2, 2), (65535, 3, 33, 32, 2, 2)])
def test_full_precision_keys_beside_packed_ones(recorder, b, h, n, r, dt, launches, pc):
    got = recorded.run(recorder, CODE % dict(b=b, h=h, n=n, r=r, pc=pc, dt=dt))
    assert got["rc"] == 0 and len(got["grids"]) == launches
    tail, es = n % r, 4 if dt == 0 else 2
    eights = (tail + 7) // 8
    assert launches == 1 + (b * h * eights * 8 * 128 * es > 24 << 20)
    x, y, z = got["grids"][0]
    if launches == 1:                                     # a row per head, and wavefronts (four a workgroup) for the tail behind
        assert z == 1 and y <= 65535 and x * (y - b * h) * 4 >= b * h * eights > (x * (y - b * h) - x) * 4 - 4
    else:
        assert y * z == b * h


@pytest.mark.parametrize("bits,group", [(2, 32), (2, 128), (4, 32), (4, 64)])
def test_workgroups_of_the_packed_keys(recorder, bits, group):
    """A launch is spread over the chip as far as its workgroups are resident together: 4 bits in groups of 32 leave room for
    three per CU, the others for four."""
    shapes = [(b, n) for b in (1, 4, 8, 16, 64, 100, 512) for n in (33, 512, 1000, 1024, 4096, 8192, 32768)]
    code = """
out = []
for b, n in %r:
    n0 = rec.recorded()
    assert lib.squat_key_scores(0x10000, 0x20000, 0x30000, b, 8, n, 128, %d, %d, 0x40000, 2, 4, 8 * 4 * 128, 128, 1.0, 0x50000,
                                8 * 4 * n, n, None) == 0
    assert rec.recorded() == n0 + 1
    out.append(list(rec.launch_at(n0).contents.grid))
print(json.dumps(out))
""" % (shapes, bits, group)
    aim = 512 if (bits, group) == (4, 32) else 1024
    for (b, n), (x, y, z) in zip(shapes, recorded.run(recorder, code)):
        units = -(-n // 16)
        assert (y, z) == (8 * b, 1) and x * y <= max(1.5 * aim, 1.5 * units * y / (4 * 32) + y)
        if units * y <= 4 * 32 * aim:                     # less work than fills the chip with full wavefronts
            assert x * y <= 1.5 * aim or x == 1
            assert x * y >= min(aim / 2, units * y // 8)  # (down to a pair of units a wavefront)
