"""Which stores the dequantize kernels are launched with: non-temporal ones for large outputs whose rows are whole 128-byte lines, or
begin on half lines with room between them; ordinary ones where a line is shared by two rows, and for small outputs.  A call is launched
with the same kernel as a small one, or with its twin.  Host side only, against a recorder of the launches."""
import pytest

from . import recorded

CODE = """
vp, i64, i = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
f = %s
f.argtypes = [vp, vp, vp, i64, i, i64, i, i, i, vp, i, i64, i64, i64, vp]
def launched(heads, n, base, strides):
    n0 = rec.recorded()
    assert f(0x10000, 0x20000, 0x30000, 2, heads, n, 128, %d, 32, 0x40000000 + base, %d, *strides, None) == 0 and rec.recorded() == n0 + 1
    return rec.launch_at(n0).contents.func
small = launched(8, 32, 0, (8 * 32 * 128, 32 * 128, 128))
out = []
for heads, n, base, strides in %r:
    out.append(launched(heads, n, base, strides) != small)
print(json.dumps(out))
"""


def _heads_first(heads, n, row):
    return (heads * n * row, n * row, row)


def _tokens_first(heads, n, row):
    return (heads * n * row, row, heads * row)


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return recorded.build(str(tmp_path_factory.mktemp("recorder")))


@pytest.mark.parametrize("dtype", [0, 1, 2])
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("name", ["lib.squat_dequantize_keys", "lib.squat_dequantize_keys_per_channel"])
def test_rows_that_share_lines_are_written_by_ordinary_stores(recorder, name, bits, dtype):
    n, line, es = 4096, 64 if dtype else 32, 2 if dtype else 4           # a line's elements
    cases = [(True, 0, _heads_first(8, n, 128)), (True, 128, _heads_first(8, n, 128)), (True, 0, _heads_first(8, n, 128 + line)),
             (True, 0, _tokens_first(8, n, 128)), (True, 0, _heads_first(8, n, 128 + line // 2)), (True, 64, _heads_first(8, n, 128 + line // 2)),
             (True, 64, _heads_first(8, n, 128 + line)), (True, 0, (8 * n * 128 + line, n * 128 + line, 128)),
             (False, 16, _heads_first(8, n, 128)), (False, 64, _heads_first(8, n, 128)), (False, 64, _tokens_first(8, n, 128)),
             (False, 0, _heads_first(8, n, 136)), (False, 32, _heads_first(8, n, 128 + line)), (False, 0, (8 * n * 128 + 8, n * 128, 128)),
             (False, 0, (8 * n * 128, n * 128 + 8, 128))]
    got = recorded.run(recorder, CODE % (name, bits, dtype, [(8, n, b, s) for _, b, s in cases]))
    assert got == [want for want, _, _ in cases]
    # from 4 MB on; strides over a single head do not count
    rows = (4 << 20) // (128 * es) // 2                                  # of each of two batch entries
    sizes = [(1, rows, 0, (rows * 128, 8, 128)), (1, rows - 32, 0, (rows * 128, 8, 128)), (rows // 32, 32, 0, _heads_first(rows // 32, 32, 128))]
    assert recorded.run(recorder, CODE % (name, bits, dtype, sizes)) == [True, False, True]


@pytest.mark.parametrize("dtype", [0, 1, 2])
@pytest.mark.parametrize("per_channel", [False, True])
def test_large_outputs(recorder, per_channel, dtype):
    """Per channel whole lines are streamed up to 512 MB (fp32 256 MB), per token and half lines whatever the size."""
    name = "lib.squat_dequantize_keys" + ("_per_channel" if per_channel else "")
    n, pad = 1 << 17, 32 if dtype else 16
    sizes = [(8, n, 0, _heads_first(8, n, 128)), (8, n + 32, 0, _heads_first(8, n + 32, 128)), (8, n + 32, 0, _heads_first(8, n + 32, 128 + pad))]
    assert dtype == 0 or 2 * 8 * n * 256 == 512 << 20
    if dtype == 0:
        sizes = [(8, n // 4, 0, _heads_first(8, n // 4, 128)), (8, n // 4 + 32, 0, _heads_first(8, n // 4 + 32, 128)), sizes[2]]
        assert 2 * 8 * (n // 4) * 512 == 256 << 20
    assert recorded.run(recorder, CODE % (name, 2, dtype, sizes)) == [True, not per_channel, True]
