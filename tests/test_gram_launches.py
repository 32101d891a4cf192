"""How a Gram matrix is split among workgroups (one fills a compute unit: a launch of more than 256 would run in two rounds, which
only head counts above 128 do) and which kernel sums the partial matrices.  Host side only, against a recorder of the launches; the sums themselves:
test_gpu_gram_split.py."""
import pytest

from . import recorded

CUS, WAVES = 256, 4
F32, BF16 = 0, 2

CODE = """
out = []
for dt, n, heads, qpk in %r:
    ws = lib.squat_build_subspace_workspace(n, heads, qpk, 128, 0)
    n0 = rec.recorded()
    assert lib.squat_build_subspace(0x10000, dt, n, heads, qpk, 128, n * 128, 128, 0, None, None, None, 0x100000, ws, None) == 0
    assert rec.recorded() == n0 + 2
    out.append([list(rec.launch_at(n0 + i).contents.grid) + [rec.launch_at(n0 + i).contents.shared] for i in range(2)])
print(json.dumps(out))
"""


@pytest.fixture(scope="module")
def grids(tmp_path_factory):
    shapes = [(dt, n, heads, qpk) for dt in (F32, BF16) for n in (1, 16, 130, 200, 512, 1024, 4096) for qpk in (1, 4)
              for heads in (1, 2, 4, 7, 8, 12, 16, 17, 20, 24, 25, 28, 31, 32, 33, 36, 40, 48, 64, 65, 85, 86, 96, 127, 128, 129, 200, 300)]
    rec = recorded.build(str(tmp_path_factory.mktemp("recorder")))
    return dict(zip(shapes, recorded.run(rec, CODE % (shapes,))))


def test_workgroups_per_head(grids):
    for (dt, n, heads, qpk), (gram, _) in grids.items():
        wgs, rest = divmod(gram[0], heads)
        assert rest == 0 and wgs >= 1
        chunks = qpk * -(-n // 16)
        eight, two = -(-chunks // (8 * WAVES)), -(-chunks // (2 * WAVES))        # chunks per wavefront
        held = CUS // heads                               # of a head, all heads' at once
        room = held if held > 1 else -(-CUS // heads)
        assert wgs <= room and wgs <= two
        assert wgs >= min(eight, room)
        if wgs > min(eight, room):                        # the finer split: within one round, 16-bit only for few workgroups
            assert wgs * heads <= CUS
            assert dt == F32 or heads * eight <= 16
        if dt == F32:
            assert wgs == min(eight, room) or wgs == min(two, held)


def test_kernel_of_the_reduction(grids):
    for (dt, n, heads, qpk), (gram, reduce) in grids.items():
        wgs = gram[0] // heads
        spread = wgs >= 4 or heads <= (24 if wgs == 1 else 32)
        assert reduce[:3] == ([40, heads, 1] if spread else [heads, 1, 1])


def test_longer_sums_are_made_of_two(grids):
    """A head with fewer workgroups than the number rounded up has longer sums than that number's: each wavefront then puts its first
    half's aside, all of a compute unit's 160 KB of LDS for four of them."""
    for (dt, n, heads, qpk), (gram, _) in grids.items():
        rounded_up = min(-(-qpk * -(-n // 16) // (8 * WAVES)), -(-CUS // heads))
        assert gram[3] == (160 if gram[0] // heads < rounded_up else 80) * 1024
