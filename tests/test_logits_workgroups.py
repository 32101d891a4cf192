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


@pytest.mark.parametrize("name,qpk,line", [(ROPE, 1, 3072), (ROPE, 4, 3072), (ROPE, 8, 3072), (PC_ROPE, 1, 3072), (PC_ROPE, 4, 3072), (PC_ROPE, 8, None),
                                           (PC, 1, None), (PC, 4, None), (PC, 8, 1536)])
def test_third_workgroup_of_long_sequences(recorder, name, qpk, line):
    """512 divided by 171 to 204 sequences is nearer to three than to two."""
    lengths = (512, 1024, 1536 - 64, 1536, 3072 - 64, 3072, 4096)
    cases = [(h, n) for h in (170, 171, 190, 204, 205, 256) for n in lengths]
    want = [3 if h <= 170 or (h <= 204 and line and n >= line) else 2 for h, n in cases]
    want = [min(w, -(-n // 256)) for w, (_, n) in zip(want, cases)]          # 64 tokens a wavefront at least
    assert _workgroups(recorder, name, qpk, cases) == want


@pytest.mark.parametrize("name", [ROPE, PC_ROPE])
def test_rotary_sequences_in_halves(recorder, name):
    """Of more than 384 sequences only those of more than 12 epochs of 64 tokens."""
    cases = [(h, n) for h in (257, 384, 385, 512, 513, 640, 641, 769, 896, 897, 1100) for n in (512, 768, 800, 2560)]
    want = [2 if h <= 384 or (n > 768 and (513 <= h <= 640 or 769 <= h <= 896)) else 1 for h, n in cases]
    assert _workgroups(recorder, name, 4, cases) == want
