"""Small logits outputs are written by ordinary stores also where their rows begin on 64-byte lines: below 1 MiB (per-token store
without rotary: 2 MiB) such a call is launched with the kernel that rows off the lines get, from there on with another one."""
import pytest

from . import recorded
from .test_logits_stores import CODE


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return recorded.build(str(tmp_path_factory.mktemp("recorder")))


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("qpk", [1, 4, 8])
@pytest.mark.parametrize("name,limit", [("squat_key_scores_rope", 1), ("squat_key_scores_per_channel", 1), ("squat_key_scores", 2)])
def test_line(recorder, name, limit, bits, qpk):
    n = limit * 2 ** 20 // (4 * 8 * qpk)
    shapes = [(1, 1, qpk, 32), (1, 8, qpk, 32), (1, 8, qpk, n - 32), (1, 8, qpk, n), (8, 1, qpk, n - 32), (8, 1, qpk, n)]
    code = CODE.replace("lib.squat_key_scores_rope", "lib.squat_key_scores.argtypes = lib.squat_key_scores_per_channel.argtypes\n"
                        "lib.squat_key_scores_rope")
    got = recorded.run(recorder, code % ((name, bits, name.endswith("rope")), shapes))
    assert got == [True, True, True, False, True, False]
