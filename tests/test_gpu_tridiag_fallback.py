"""Heads whose tridiagonal result does not stand on its own, beside heads that are not concerned: more than 32 directions, the 33rd
eigenvalue not below the 32nd.  Against float64: eigenvalues and the orthogonality of Qhat's rows to the rounding of the fp32
output and Gram sums (1e-6 of the largest eigenvalue), and where the directions are unique the projector.  With up to 32 directions
the same inputs stand on their own."""
import pytest
import torch

from paper_2503_24358_amd import squat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [16, 32, 33, 40, 64])
def test_ties_and_rank_deficiency_beside_ordinary_heads(r):
    gen = torch.Generator(device="cuda").manual_seed(r)
    q = torch.zeros(4, 512, 128, device="cuda")
    q[0] = torch.randn(512, 128, device="cuda", generator=gen) * 0.95 ** torch.arange(128, device="cuda")
    q[1, :20] = torch.randn(20, 128, device="cuda", generator=gen)                  # 20 directions, then nothing
    q[2, :128] = 3.0 * torch.eye(128, device="cuda")                               # every direction alike
    q[3] = torch.randn(512, 128, device="cuda", generator=gen)
    qhat, eig, _ = squat.build_subspace(q, 1, r)
    together = (qhat.clone(), eig.clone())
    x = q.double()
    gram = (x.transpose(1, 2).contiguous() @ x).cpu()
    val, vec = torch.linalg.eigh(gram)
    val, vec = val.flip(-1)[:, :r], vec.flip(-1)[:, :, :r]
    qhat, eig = qhat.double().cpu(), eig.double().cpu()
    for h in range(4):
        top = val[h, 0].item()
        assert (eig[h] - val[h]).abs().max().item() <= 1e-6 * top
        assert (qhat[h] @ qhat[h].T - torch.diag(eig[h])).abs().max().item() <= 2e-6 * top
        assert (gram[h] @ qhat[h].T - qhat[h].T * eig[h]).abs().max().item() <= 2e-6 * top * top ** 0.5
    for h in (0, 3):
        want = (vec[h] * val[h]) @ vec[h].T
        assert torch.linalg.norm(qhat[h].T @ qhat[h] - want).item() <= 1e-3 * torch.linalg.norm(want).item()
