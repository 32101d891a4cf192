"""Workgroups of a sequence in the launches of the rotary and the per-channel logits.  As many as make no more than 512, two per CU; from
257 sequences on two where the CUs with most of them then have half a sequence less to do.  Host side only, against a recorder of
the launches."""
import pytest

from . import recorded

GRIDS = """
i64, vp, ci = ctypes.c_int64, ctypes.c_void_p, ctypes.c_int
tail = [vp, ci, ci, i64, i64, ctypes.c_float, vp, i64, i64, vp]
out = []
for name, qpk, h, n in %r:
    rope = "rope" in name
    f = getattr(lib, name)
    f.argtypes = [vp, vp, vp, i64, ci, i64, ci, ci, ci] + ([vp, i64] if rope else []) + tail
    n0 = rec.recorded()
    freq = (0x60000, 3) if rope else ()
    assert f(0x10000, 0x20000, 0x30000, 1, h, n, 128, 2, 32, *freq, 0x40000, 2, qpk, h * qpk * 128, 128, 1.0, 0x50000, h * qpk * n, n, None) == 0
    out.append(list(rec.launch_at(n0).contents.grid))
print(json.dumps(out))
"""
PC, ROPE, PC_ROPE = "squat_key_scores_per_channel", "squat_key_scores_rope", "squat_key_scores_rope_per_channel"


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return recorded.build(str(tmp_path_factory.mktemp("recorder")))


def _workgroups(recorder, name, qpk, cases):
    got = recorded.run(recorder, GRIDS % ([(name, qpk, h, n) for h, n in cases],))
    assert all(g[1:] == [h, 1] for g, (h, _) in zip(got, cases))
    return [g[0] for g in got]


@pytest.mark.parametrize("qpk", [1, 4, 8])
def test_per_channel_sequences_in_halves(recorder, qpk):
    cases = [(h, n) for h in (257, 300, 341, 342, 384, 385, 512, 513, 600, 1100) for n in (512, 1024, 2560)]
    assert _workgroups(recorder, PC, qpk, cases) == [2 if h <= 384 else 1 for h, _ in cases]
