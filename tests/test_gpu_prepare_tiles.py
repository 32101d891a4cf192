"""The update matrix by block elimination at subspace sizes around its tiles (16 directions) and pivot blocks (4), against
the float64 oracle: all panels, both stored forms, a lambda that makes the matrix badly conditioned but not flagged.

Bound: the solver works in fp64; with pivots that span up to 1e9 it may lose nine of its sixteen digits, so the stored
fp32 numbers are good to 2^-24 (rounding) + 1e-7, the fp16 grid to 2^-11 per entry."""
import numpy as np
import pytest
import torch

from oracle import squat_oracle as O
from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g", [32, 64])
@pytest.mark.parametrize("r", [1, 3, 4, 5, 15, 16, 17, 20, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("lam", [1e-3, 1.0])
def test_update_matrix_at_tile_edges(r, g, lam):
    heads = 3
    rng = np.random.default_rng(r * 100 + g)
    # rows of very different size: singular values from 0.03 to 300
    q = rng.standard_normal((heads, r, 128)) * 10.0 ** rng.uniform(-2.5, 1.5, (heads, r, 1))
    qhat = q.astype(np.float32)
    t = torch.from_numpy(qhat).cuda()
    full = squat.prepare(t, lam, g, full_precision=True).cpu().numpy().astype(np.float64)
    grid = squat.prepare(t, lam, g).cpu().numpy().astype(np.float64)
    for h in range(heads):
        want = O.update_matrix_lowrank(qhat[h].astype(np.float64), lam, g)
        assert np.linalg.norm(full[h] - want) <= 2e-7 * np.linalg.norm(want)
        assert np.all(np.abs(grid[h] - full[h]) <= 2.0 ** -11 * np.abs(full[h]) + 2.0 ** -25)
        assert np.array_equal(full[h] == 0, want == 0)
