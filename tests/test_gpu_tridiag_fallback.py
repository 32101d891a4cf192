"""Heads whose tridiagonal result does not stand on its own, beside heads that are not concerned.  Against float64: eigenvalues and the
orthogonality of Qhat's rows to the rounding of the fp32 output and Gram sums (1e-6 of the largest eigenvalue), and where the
directions are unique the projector.

With more than 32 directions a 33rd eigenvalue not below the 32nd is such a case.  With up to 32 no input is known: those heads
are made by a build of the library whose solver refuses matrices of which the largest entry has an odd exponent."""
import ctypes
import math
import os

import pytest
import torch

from paper_2503_24358_amd import build, squat

pytestmark = pytest.mark.gpu


def _queries(seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q = torch.zeros(6, 512, 128, device="cuda")
    q[0, :256] = torch.randn(256, 128, device="cuda", generator=gen) * 0.95 ** torch.arange(128, device="cuda")
    q[1, :20] = torch.randn(20, 128, device="cuda", generator=gen)                  # 20 directions, then nothing
    q[2, :128] = 3.0 * torch.eye(128, device="cuda")                               # every direction alike
    q[3, :256] = torch.randn(256, 128, device="cuda", generator=gen)
    q[4, :128] = torch.diag(torch.arange(128, 0, -1, device="cuda").float())       # a diagonal Gram matrix (and the last head: zero)
    return q


TIES, UNIQUE = (1, 2), (0, 3, 4)


def _build_subspace(call, q, r):
    """(Qhat, eigenvalues, which heads were redone: the library keeps one int a head in the last block of its workspace)."""
    heads, n, _ = q.shape
    nbytes = squat.build_subspace_workspace(n, heads, 1, 128, r)
    ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    qhat, eig = torch.empty(heads, r, 128, device="cuda"), torch.empty(heads, r, device="cuda")
    p = [ctypes.c_void_p(t.data_ptr()) for t in (q, qhat, eig, ws)]
    assert call(p[0], squat.F32, n, heads, 1, 128, n * 128, 128, r, p[1], p[2], None, p[3], nbytes,
                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    marks = ws[nbytes - (4 * heads + 255) // 256 * 256:].view(torch.int32)[:heads].tolist()
    return qhat, eig, marks


def _check(gram, r, qhat, eig, unique):
    val, vec = torch.linalg.eigh(gram)
    val, vec = val.flip(-1)[:, :r], vec.flip(-1)[:, :, :r]
    qhat, eig = qhat.double().cpu(), eig.double().cpu()
    for h in range(len(gram)):
        top = val[h, 0].item()
        assert (eig[h] - val[h]).abs().max().item() <= 1e-6 * top
        assert (qhat[h] @ qhat[h].T - torch.diag(eig[h])).abs().max().item() <= 2e-6 * top
        assert (gram[h] @ qhat[h].T - qhat[h].T * eig[h]).abs().max().item() <= 2e-6 * top * top ** 0.5
    for h in unique:
        want = (vec[h] * val[h]) @ vec[h].T
        assert torch.linalg.norm(qhat[h].T @ qhat[h] - want).item() <= 1e-3 * torch.linalg.norm(want).item()


def _gram(q):
    x = q.double()
    return (x.transpose(1, 2).contiguous() @ x).cpu()


@pytest.mark.parametrize("r", [16, 32, 33, 40, 64])
def test_ties_and_rank_deficiency_beside_ordinary_heads(r):
    q = _queries(r)
    qhat, eig, marks = _build_subspace(squat.lib().squat_build_subspace, q, r)
    assert marks == [int(r > 32 and h in TIES) for h in range(6)]
    _check(_gram(q), r, qhat, eig, UNIQUE)
    for h in range(len(q)):                                # a head's result does not depend on the others'
        alone = _build_subspace(squat.lib().squat_build_subspace, q[h:h + 1], r)
        assert torch.equal(alone[0][0], qhat[h]) and torch.equal(alone[1][0], eig[h]) and alone[2] == marks[h:h + 1]


@pytest.fixture(scope="module")
def refusing():
    lib = ctypes.CDLL(build.REFUSING_LIB if os.path.exists(build.REFUSING_LIB) else build.build_refusing())
    lib.squat_build_subspace.argtypes = squat.lib().squat_build_subspace.argtypes
    return lib.squat_build_subspace


@pytest.mark.parametrize("r", [1, 8, 16, 31, 32, 40])
def test_refused_heads_beside_accepted_ones(refusing, r):
    q = _queries(100 + r)
    q = torch.cat([q, q])
    q[6:, 256:] = q[6:, :256]                              # every token twice: the Gram matrix doubled, the exponent one higher
    gram = _gram(q)
    odd = [h % 6 < 5 and math.frexp(gram[h].abs().max().item())[1] % 2 == 0 for h in range(12)]      # (frexp's is one higher)
    assert sum(odd) == 5
    qhat, eig, marks = _build_subspace(refusing, q, r)
    assert marks == [int(odd[h] or (r > 32 and h % 6 in TIES)) for h in range(12)]
    _check(gram, r, qhat, eig, [h for h in range(12) if h % 6 in UNIQUE])
    want = _build_subspace(squat.lib().squat_build_subspace, q, r)
    for h in range(12):
        if not marks[h]:
            assert torch.equal(qhat[h], want[0][h]) and torch.equal(eig[h], want[1][h])
