"""squat_cache_append may be repeated after an error: whatever launch of it failed, the values have been touched (the oldest
one quantized, its ring slot overwritten) only if the counters say so.  Host side only, against a recorder of the launches."""
import pytest

from . import recorded


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return recorded.build(str(tmp_path_factory.mktemp("recorder")))


# The append kernel's first two parameter words are its key and value pointers; a launch with a value pointer writes the
# ring.  After `before` tokens the next append is made to fail at its launch `bad` (None: an error of an earlier, unrelated
# call is pending), then repeated.
CODE = """
h = R.cache(lib, residual=%(residual)d, quantize_values=%(values)d, key_per_channel=%(pc)d, max_tokens=256)
K, V = 0x10000, 0x20000
append = lambda: lib.squat_cache_append(h, K, V, 3 * 128, 128, None)
for _ in range(%(before)d): assert append() == 0
kernel = rec.launch_at(0).contents.func
old, n0 = R.counts(lib, h), rec.recorded()
bad = %(bad)r
if bad is None: rec.leave_error(2)
else: rec.fail_launch(n0 + bad)
first = append()
mid = R.counts(lib, h)
rec.fail_launch(-1)
second = append()
ran = [rec.launch_at(i).contents for i in range(n0, rec.recorded())]
ran = [l for l in ran if not l.failed]
print(json.dumps(dict(first=first, second=second, old=old, mid=mid, new=R.counts(lib, h),
                      keys=sum(l.func == kernel and l.head[0] == K for l in ran),
                      values=sum(l.func == kernel and l.head[1] == V for l in ran),
                      flushes=sum(l.func != kernel for l in ran))))
"""


@pytest.mark.parametrize("residual,before,pc,bad",                     # the token that fills the key buffer: three launches
                         [(r, n, pc, bad) for r, n, pc in ((4, 11, 0), (4, 3, 0), (32, 63, 1), (4, 9, 0), (4, 2, 0))
                          for bad in (None, 0, 1, 2)[:4 if (n + 1) % r == 0 else 2]])
def test_a_failed_append_can_be_repeated(recorder, residual, before, pc, bad):
    flush = (before + 1) % residual == 0
    r = recorded.run(recorder, CODE % dict(residual=residual, values=1, pc=pc, before=before, bad=bad))
    assert r["first"] != 0 and r["mid"] == r["old"]
    assert r["second"] == 0
    assert r["new"][0] == before + 1
    assert r["new"][1:3] == [(before + 1) // residual * residual, (before + 1) % residual]
    assert r["values"] == 1                               # the new value went to the ring once
    assert r["keys"] >= 1 and (r["flushes"] >= 1) == flush


@pytest.mark.parametrize("before", [2, 3])
def test_keys_alone(recorder, before):
    r = recorded.run(recorder, CODE.replace("K, V =", "V = None; K, _ =") % dict(residual=4, values=0, pc=0, before=before, bad=0))
    assert r["first"] != 0 and r["mid"] == r["old"] and r["second"] == 0 and r["new"][0] == before + 1 and r["keys"] == 1
