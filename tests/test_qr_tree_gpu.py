"""The TSQR tree's two schedules and the WY kernels at the edges of their tiles.

A workspace of the size the size function asks for lets the levels of the tree
pass on R before any Q is formed; one a byte shorter runs the levels one after
the other.  Both apply the same reflections and form Q by the same products, so
Q and R agree bit for bit.

Y = W (I - Q_1)^-1: with the inverse M exact and then rounded, the stored W, n
products accumulated in FP32 and the rounding of the result, an entry of Y is
off by at most (n + 4) u (|W| |M|) with u = 2^-24; the FP64 elimination itself
is far below that.
"""
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


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to("cuda")


@pytest.mark.parametrize("shape", [(257, 1), (600, 64), (1030, 63), (5000, 33), (70000, 64)])
@pytest.mark.parametrize("pad", [0, 3])
def test_tsqr_schedules_agree(la, shape, pad):
    m, n = shape
    buf = dev(la_inputs.gaussian((m, n + pad), 900 + m + n))
    A = buf[:, :n]
    size = int(la.lib().la_tsqr_workspace_size(m, n))
    Q, R = la.tsqr(A, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
    Q1, R1 = la.tsqr(A, workspace=torch.empty(size - 1, dtype=torch.uint8, device="cuda"))
    assert torch.equal(R, R1) and torch.equal(Q, Q1)
    assert torch.isfinite(Q).all()


@pytest.mark.parametrize("shape,panel", [((700, 300), 64), ((1100, 129), 33), ((900, 260), 7)])
def test_caqr_schedules_agree(la, shape, panel):
    A = dev(la_inputs.gaussian(shape, 930 + panel))
    size = la.caqr_workspace_size(*shape, panel, True)
    Q, R = la.caqr(A, panel=panel, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
    Q1, R1 = la.caqr(A, panel=panel,
                     workspace=torch.empty(size - 1, dtype=torch.uint8, device="cuda"))
    assert torch.equal(R, R1) and torch.equal(Q, Q1)


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 31, 63, 64, 65, 100, 127, 128])
@pytest.mark.parametrize("extra", [50, 1500])   # square: 1 can be an eigenvalue of Q
def test_wy_edges(la, n, extra):
    m = n + extra
    Q, _ = np.linalg.qr(la_inputs.gaussian((m, n), 960 + n + extra).astype(np.float64))
    Q32 = Q.astype(np.float32)
    W, Y = la.wy(dev(Q32))
    torch.cuda.synchronize()
    W, Y = W.cpu().numpy().astype(np.float64), Y.cpu().numpy().astype(np.float64)
    W0 = (Q32 - np.eye(m, n, dtype=np.float32)).astype(np.float32)
    assert np.array_equal(W, W0.astype(np.float64))
    M = np.linalg.inv(np.eye(n) - Q32[:n].astype(np.float64))
    bound = (n + 4) * 2.0 ** -24 * (np.abs(W) @ np.abs(M))
    assert np.all(np.abs(Y - W @ M) <= bound + 1e-30)
