"""The exact eigen-solver behind squat_build_subspace on Gram matrices given directly (squat_refresh_subspace with
iterations < 0 solves the state it holds): spectra with gaps on both sides of the solver's 1e-11 rule (twisted
factorisation or inverse iteration), coincident and vanishing eigenvalues, nearly diagonal and decoupled matrices, and
subspace sizes at the edges of its thread teams and batches.

Bounds: a row is sqrt(lambda) v rounded to fp32, off by at most 2^-24 of its norm in the 2-norm, and the solver accepts
vectors whose residual and orthogonality are good to 1e-9, so products of two normalised rows and residuals are within
2 * 2^-24 + 1e-9 < 1.3e-7; for rows with a small lambda (kept down to 1e-5 of the largest singular value) the
residual is relative to the largest eigenvalue.  The tests allow 1.5e-7."""
import numpy as np
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu

D = 128


def _spectrum(kind):
    i = np.arange(D)
    return {"decay": 0.9 ** i * 1e4, "gaps_1e-5": 100 * (1 - 1e-5 * i), "gaps_1e-9": 100 * (1 - 1e-9 * i),
            "gaps_3e-11": 100 * (1 - 3e-11 * i), "gaps_1e-12": 100 * (1 - 1e-12 * i),
            "coincident": np.where(i < 20, 5.0, 1.0), "equal": np.full(D, 3.0), "rank_12": np.maximum(12.0 - i, 0.0),
            "graded": 10.0 ** (-i / 8.0)}[kind]


def _matrix(kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "identity":
        return np.eye(D)
    if kind == "diagonal":
        return np.diag(np.arange(D, 0, -1.0))
    if kind == "tridiagonal":                  # pairs of eigenvalues that agree to the last bits
        return np.diag(np.abs(i := np.arange(D) - 63.5) + 2) + np.diag(np.ones(D - 1), 1) + np.diag(np.ones(D - 1), -1)
    if kind == "blocks":                       # decoupled, each block's eigenvalues repeated eight times
        x = rng.standard_normal((16, 16))
        return np.kron(np.eye(8), x @ x.T)
    q, _ = np.linalg.qr(rng.standard_normal((D, D)))
    g = (q * _spectrum(kind)) @ q.T
    return (g + g.T) / 2


@pytest.mark.parametrize("r", [1, 5, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("kind", ["decay", "gaps_1e-5", "gaps_1e-9", "gaps_3e-11", "gaps_1e-12", "coincident", "equal",
                                  "rank_12", "graded", "identity", "diagonal", "tridiagonal", "blocks"])
def test_exact_solver_on_given_matrices(kind, r):
    heads = 3
    g = np.stack([_matrix(kind, 40 + h) * 10.0 ** (4 * h - 4) for h in range(heads)])
    qhat, eig, _ = squat.refresh_subspace(torch.from_numpy(g).cuda(), 1, r, -1)
    qhat, eig = qhat.cpu().numpy().astype(np.float64), eig.cpu().numpy().astype(np.float64)
    for h in range(heads):
        lam = np.maximum(np.linalg.eigvalsh(g[h])[::-1][:r], 0.0)
        assert np.abs(eig[h] - lam).max() <= 1.5e-7 * lam[0]
        keep = lam > 1e-10 * lam[0]
        x = qhat[h][keep] / np.sqrt(lam[keep])[:, None]
        n = len(x)
        tol = 1.5e-7 + 1e-15 * lam[0] / lam[keep].min()       # (numpy's own lambda: 1e-15 of the largest)
        assert np.abs(x @ x.T - np.eye(n)).max() <= tol, (h, np.abs(x @ x.T - np.eye(n)).max())
        assert np.linalg.norm(g[h] @ x.T - x.T * lam[keep], axis=0).max() <= 1.5e-7 * lam[0]
        # the largest component is positive (one that is equally large but for the rounding may be negative)
        assert (x.max(axis=1) >= np.abs(x).max(axis=1) - 1.5e-7).all()
