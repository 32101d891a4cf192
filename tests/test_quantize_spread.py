"""How a quantize launch is spread: the workgroups of all problems (update matrices) fit the device at once, since one that waits
for another to end doubles the time of a launch, and the plan query tells what is launched.  The grids on the host, against a recorder of the launches, for every number
of heads; the launch on the GPU."""
import pytest
import torch

from paper_2503_24358_amd import squat

from . import recorded

CUS = 256          # planned for without a GPU, and an MI355X's

CODE = """
vp, i64, i = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
class Plan(ctypes.Structure):
    _fields_ = [("problems", i64), ("workgroups", i), ("wavefronts", i), ("tiles", i64)]
lib.squat_quantize_keys_plan.argtypes = [i, i64, i, i64, i, i64, i, i, i, i, vp]
out = []
for per_channel, f in enumerate((lib.squat_quantize_keys, lib.squat_quantize_keys_per_channel)):
    f.argtypes = [vp, i, i64, i, i64, i, i64, i64, i64, vp, i64, i, i, i, vp, vp, vp, vp]
    for heads, n in %r:
        n0 = rec.recorded()
        assert f(0x10000, 2, 3, heads, n, 128, heads * n * 128, n * 128, 128, 0x20000, 0, 2, 32, 32, 0x30000, 0x40000, 0x50000, None) == 0
        assert rec.recorded() == n0 + 1
        launch, plan = rec.launch_at(n0).contents, Plan()
        assert lib.squat_quantize_keys_plan(2, 3, heads, n, 1, 0, 2, 32, 32, per_channel, ctypes.byref(plan)) == 0
        out.append([list(launch.grid), launch.block[0], plan.problems, plan.workgroups, plan.wavefronts, plan.tiles])
print(json.dumps(out))
"""


def test_workgroups_fit_the_device(tmp_path):
    shapes = [(heads, n) for heads in list(range(1, 258)) + [300, 512, 1024] for n in (32, 96, 4096)]
    grids = recorded.run(recorded.build(str(tmp_path)), CODE % (shapes,))
    for (heads, n), (grid, threads, *plan) in zip(2 * shapes, grids):
        wgs, rest = divmod(grid[0], heads)
        tiles = 3 * (n // 32)
        assert plan == [heads, wgs, threads // 64, tiles]
        assert rest == 0 and grid[1:] == [1, 1] and 1 <= wgs <= tiles
        assert grid[0] <= max(CUS, heads)
        assert wgs == tiles or grid[0] + heads > CUS          # and no fewer than fit


@pytest.mark.gpu
@pytest.mark.parametrize("heads,n", [(3, 4100), (7, 1000), (130, 96), (257, 40)])
@pytest.mark.parametrize("per_channel", [False, True])
def test_heads_that_do_not_divide_the_device(heads, n, per_channel):
    """A head's words do not depend on the other heads of the launch."""
    gen = torch.Generator(device="cuda").manual_seed(heads)
    n = n // 32 * 32 if per_channel else n
    k = torch.randn(2, heads, n, 128, device="cuda", generator=gen).to(torch.bfloat16)
    u = torch.randn(heads, 128, 128, device="cuda", generator=gen).mul(0.05).tril(-1).half().float()
    f = squat.quantize_keys_per_channel if per_channel else squat.quantize_keys
    together = f(k, u, 2, 32, 32)
    for h in {0, heads // 2, heads - 1}:
        alone = f(k[:, h:h + 1].contiguous(), u[h:h + 1].contiguous(), 2, 32, 32)
        for a, b in zip(together, alone):
            assert torch.equal(a[:, h:h + 1], b)
