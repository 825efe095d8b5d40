"""TSQR of 65 to 128 columns: the factors of every level go ahead and all blocks'
Q follow in one launch, from the reflectors and kappa left in Q's place.

Backward error and orthogonality as for the narrower panels: a reflection commits
a few u = 2^-24 per element and an element passes n of them per level, so with
L levels both stay below 4 sqrt(n (L + 1)) u."""
import math

import numpy as np
import pytest
import torch

import la_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


@pytest.mark.parametrize("m,n", [(65, 65), (128, 128), (255, 127), (257, 72), (300, 128),
                                 (384, 65), (513, 121), (2049, 100), (40000, 128)])
@pytest.mark.parametrize("pad", [0, 3])
def test_wide_tsqr(la, m, n, pad):
    buf = torch.from_numpy(la_inputs.gaussian((m, n + pad), 970 + m + n)).cuda()
    A = buf[:, :n]
    Q, R = la.tsqr(A)
    torch.cuda.synchronize()
    A, Q, R = A.double(), Q.double(), R.double()
    levels, blocks = 1, -(-m // 256)
    while blocks > 1:
        levels, blocks = levels + 1, -(-blocks * n // 256)
    tol = 4 * math.sqrt(n * (levels + 1)) * 2.0 ** -24
    assert torch.all(torch.tril(R, -1) == 0)
    assert torch.linalg.norm(A - Q @ R) <= tol * torch.linalg.norm(A)
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    assert torch.linalg.norm(Q.T @ Q - eye) <= tol * math.sqrt(n)


def test_wide_zero_columns(la):
    """A zero column takes no reflection (kappa = 0), the first one included."""
    A = la_inputs.gaussian((700, 90), 991)
    A[:, 0] = 0.0
    A[:, 2] = 0.0
    A[:, 89] = 0.0
    Q, R = la.tsqr(torch.from_numpy(A).cuda())
    Q, R = Q.cpu().numpy().astype(np.float64), R.cpu().numpy().astype(np.float64)
    assert np.all(R[:, 0] == 0.0) and np.all(R[:, 89] == 0.0)
    assert np.linalg.norm(A - Q @ R) <= 1e-5 * np.linalg.norm(A)
    assert np.linalg.norm(Q.T @ Q - np.eye(90)) <= 1e-5 * math.sqrt(90)
