"""TSQR and WY of at most 32 columns, whose row products run on tiles of 32, at their
edges and with every kind of row stride; and the scalars of a reflection.

A - Q R and Q^T Q - I stay within the factorisations' tolerance; with u = 2^-24, W = Q - [I; 0] is one rounding, and Y is within (n + 4) u
|W| |(I - Q_1)^-1| of W (I - Q_1)^-1 entry by entry (n FP32 products and sums, the
rounding of the inverse and of W).  A column's beta is its norm by one Newton step from an
estimate within an ulp, so it is the correctly rounded square root unless that lies
within 2^-21 ulp of a tie: one in 10000 samples is allowed to."""
import math

import numpy as np
import pytest
import torch

import la_inputs

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
TOL = 1e-5


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


@pytest.mark.parametrize("n", [1, 3, 4, 8, 16, 20, 31, 32, 33])
@pytest.mark.parametrize("m", [300, 2049])
@pytest.mark.parametrize("pad", [0, 1, 4])
def test_narrow(la, m, n, pad):
    buf = torch.from_numpy(la_inputs.gaussian((m, n + pad), 950 + m + n)).cuda()
    A = buf[:, :n]
    Q, R = la.tsqr(A)
    torch.cuda.synchronize()
    A, Qd, R = A.double(), Q.double(), R.double()
    assert torch.linalg.norm(A - Qd @ R) <= TOL * torch.linalg.norm(A)
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    assert torch.linalg.norm(Qd.T @ Qd - eye) <= TOL * math.sqrt(n)

    ld = n + pad
    Qp, W, Y = (torch.full((m, ld), 5.0, device="cuda") for _ in range(3))
    Qp[:, :n] = Q
    need = int(la.lib().la_wy_workspace_size(n))
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    st = la.lib().la_wy(la.context(0), m, n, Qp.data_ptr(), ld, W.data_ptr(), ld, Y.data_ptr(), ld,
                        (ws.data_ptr() + 255) & ~255, need,
                        torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st == la.Status.OK
    for t in (W, Y):
        assert bool((t[:, n:] == 5.0).all())
    want = Q.clone()
    want[:n].diagonal().sub_(1.0)
    assert torch.equal(W[:, :n], want)
    inv = torch.linalg.inv((eye - Qd[:n]).cpu()).cuda()
    exact = want.double() @ inv
    assert torch.all((Y[:, :n].double() - exact).abs() <=
                     (n + 4) * U * (want.double().abs() @ inv.abs()) + 1e-30)


@pytest.mark.parametrize("n", [64, 128])
def test_beta_is_the_rounded_norm(la, n):
    """Columns of two entries with no row in common: each norm is formed from RN(a^2) +
    RN(b^2), and no reflection touches another column."""
    r = la_inputs.rng(77)
    off = total = 0
    for _ in range(100):
        a, b = (r.choice([-1.0, 1.0], n) * 2.0 ** r.uniform(-40, 40, n) for _ in range(2))
        b = (b * r.choice([0.0, 1e-3, 1.0], n)).astype(np.float32)
        a = a.astype(np.float32)
        A = np.zeros((256, n), np.float32)
        A[np.arange(n), np.arange(n)] = a
        A[128 + np.arange(n), np.arange(n)] = b
        _, R = la.tsqr(torch.from_numpy(A).cuda())
        want = -np.copysign(np.sqrt(a * a + b * b), a)
        got = R.diagonal().cpu().numpy()
        assert want.dtype == np.float32
        assert np.all(np.abs(got - want) <= np.spacing(np.abs(want)))
        off += int((got != want).sum())
        total += n
    assert off * 10000 <= total, off
