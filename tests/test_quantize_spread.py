"""How a quantize launch is spread: the workgroups of all problems (update matrices) fit the device at once, since one that waits
for another to end doubles the time of a launch.  The plan on the host, for every number of heads; the launch on the GPU."""
import pytest
import torch

from paper_2503_24358_amd import squat

CUS = 256          # planned for without a GPU, and an MI355X's


@pytest.mark.parametrize("per_channel", [False, True])
def test_workgroups_fit_the_device(per_channel):
    for heads in list(range(1, 258)) + [300, 512, 1024]:
        for n in (32, 96, 4096):
            p = squat.quantize_keys_plan(torch.bfloat16, 3, heads, n, True, 0, 2, 32, 32, per_channel=per_channel)
            wgs = p.problems * p.workgroups_per_problem
            assert p.problems == heads and p.tiles_per_problem == 3 * (n // 32) and 1 <= p.workgroups_per_problem <= p.tiles_per_problem
            assert wgs <= max(CUS, heads)
            # and no fewer than fit
            assert p.workgroups_per_problem == p.tiles_per_problem or wgs + heads > CUS


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
