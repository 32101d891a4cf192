"""Which stores the logits kernels are launched with: rows that begin on 64-byte lines by non-temporal ones, others by ordinary
ones except where a rule on the size of the output says otherwise.  A call whose rows are off the lines is launched with the
same kernel as one whose rows are on them, or with its twin.  Host side only, against a recorder of the launches."""
import pytest

from . import recorded


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return recorded.build(str(tmp_path_factory.mktemp("recorder")))


CODE = """
i64, vp, ci = ctypes.c_int64, ctypes.c_void_p, ctypes.c_int
tail = [vp, ci, ci, i64, i64, ctypes.c_float, vp, i64, i64, vp]
lib.squat_key_scores_per_channel.argtypes = [vp, vp, vp, i64, ci, i64, ci, ci, ci] + tail
lib.squat_key_scores_rope.argtypes = [vp, vp, vp, i64, ci, i64, ci, ci, ci, vp, i64] + tail
name, bits, rope = %r
out = []
for b, h, qpk, n in %r:
    func = []
    for width in (-(-n // 16) * 16, -(-n // 16) * 16 + 1):
        n0 = rec.recorded()
        freq = (0x60000, 3) if rope else ()
        rc = getattr(lib, name)(0x10000, 0x20000, 0x30000, b, h, n, 128, bits, 32, *freq, 0x40000, 2, qpk, h * qpk * 128, 128, 1.0, 0x50000,
                                h * qpk * width, width, None)
        assert rc == 0 and rec.recorded() == n0 + 1, rc
        func.append(rec.launch_at(n0).contents.func)
    out.append(func[0] == func[1])
print(json.dumps(out))
"""


def _shapes(mib, qpk):
    """Heads of 2048 tokens and of as many as 8 of them need, of about that much output."""
    heads = max(1, round(mib * 2 ** 20 / (4 * 2048 * qpk)))
    return [(heads, 1, qpk, 2048), (1, 8, qpk, round(mib * 2 ** 20 / (4 * 8 * qpk)) // 32 * 32)]


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("qpk", [1, 4, 8])
def test_rotary(recorder, bits, qpk):
    sizes = (1, 4, 5.5, 8, 12, 17.5, 18.5, 45)
    shapes = [s for m in sizes for s in _shapes(m, qpk)]
    got = recorded.run(recorder, CODE % (("squat_key_scores_rope", bits, True), shapes))
    assert got == [5 < m < 18 for m in sizes for _ in range(2)]


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("qpk", [1, 4, 8])
def test_per_channel(recorder, bits, qpk):
    sizes = (1, 2.25, 2.75, 3.75, 4.25, 8, 17.5, 18.5, 45)
    shapes = [s for m in sizes for s in _shapes(m, qpk)]
    got = recorded.run(recorder, CODE % (("squat_key_scores_per_channel", bits, False), shapes))
    assert got == [qpk <= 4 and (2.5 if bits == 2 else 4) < m < 18 for m in sizes for _ in range(2)]
