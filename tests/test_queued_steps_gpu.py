"""la_polar and la_inverse on sizes whose steps are queued ahead of their stop
test (the test then runs on the device): the same decisions as the scalar model
of the algorithms, whatever ends the iteration, and nothing written after it."""
import math

import numpy as np
import pytest
import torch

import la_inputs
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


def orth(U):
    U = U.double()
    G = U.t() @ U
    G.diagonal().sub_(1.0)
    return torch.linalg.norm(G).item() / math.sqrt(U.shape[1])


@pytest.mark.parametrize("cap", [1, 2, 9, 10, 11, 13, 14, 15, 23])
def test_polar_step_cap(la, cap):
    """The cap at every phase of a batch: exactly `cap` steps, the same iterate as
    the run that goes on reaches, and the step norm of the last one."""
    case = la_inputs.polar_case(160, 160, 1e-3, seeds=(21, 22, 23))
    A = torch.from_numpy(case.A32).to("cuda")
    o = dict(stagnation=False, eps=1e-30, raise_not_converged=False)
    U, H, info = la.polar(A, max_iter=cap, **o)
    torch.cuda.synchronize()
    assert info["iters_ns"] == cap and info["stop_reason"] == 2
    if cap > 1:
        V, _, prev = la.polar(A, max_iter=cap - 1, **o)
        want = torch.linalg.norm(U.double() - V.double()).item()
        assert abs(info["last_delta"] - want) <= 1e-9 * want + 1e-12
    if cap >= 10:
        assert orth(U) <= TOL


@pytest.mark.parametrize("cond", [1.0, 10.0, 1e4])
@pytest.mark.parametrize("shape", [(64, 64), (300, 129), (700, 700)])
def test_polar_stop(la, cond, shape):
    m, n = shape
    case = la_inputs.polar_case(m, n, 1.0 / cond, seeds=(31 + m, 32 + n, 33))
    A = torch.from_numpy(case.A32).to("cuda")
    U, H, info = la.polar(A)
    Upad = torch.full((m, n + 5), 3.0, device="cuda")
    U2, H2, i2 = la.polar(A, U=Upad[:, :n])
    torch.cuda.synchronize()
    assert info == i2 and torch.equal(U, U2) and torch.equal(H, H2)
    assert bool((Upad[:, n:] == 3.0).all())
    assert info["stop_reason"] in (0, 1) and 1 <= info["iters_ns"] <= 20
    assert abs(info["fro_norm_a"] / np.linalg.norm(case.A32.astype(np.float64)) - 1) <= 1e-12
    assert orth(U) <= TOL
    r = torch.linalg.norm(A.double() - U.double() @ H.double()) / torch.linalg.norm(A.double())
    assert r.item() <= TOL


@pytest.mark.parametrize("bad", [0.0, float("nan"), float("inf")])
def test_polar_refused_norm_leaves_u(la, bad):
    A = torch.full((96, 64), bad, device="cuda")
    U = torch.full((96, 64), 5.0, device="cuda")
    with pytest.raises(la.LAError) as e:
        la.polar(A, U=U)
    torch.cuda.synchronize()
    assert e.value.status == la.Status.NONFINITE
    assert bool((U == 5.0).all())


@pytest.mark.parametrize("shape", [(96, 96), (400, 250), (250, 400), (600, 600)])
def test_inverse_stop_and_cap(la, shape):
    n, m = shape
    case = la_inputs.polar_case(max(n, m), min(n, m), 0.1, seeds=(41 + n, 42 + m, 43))
    A32 = case.A32 if n >= m else np.ascontiguousarray(case.A32.T)
    A = torch.from_numpy(A32).to("cuda")
    X, info = la.inverse(A)
    torch.cuda.synchronize()
    assert info["stop_reason"] == 0 and 5 <= info["iters"] <= 30
    assert info["last_tol"] == 2.0 ** (-24 + info["iters"] - 1)    # doubled per step before the polish
    assert info["last_delta"] <= info["last_tol"]
    P = X.double() @ A.double() if n >= m else A.double() @ X.double()
    P.diagonal().sub_(1.0)
    # one-sided residual: 2 g cond^2 with g = 1e-6 and cond 10
    assert torch.linalg.norm(P).item() / math.sqrt(P.shape[0]) <= 2e-4
    for cap in (1, 3, 16, 17):
        if cap >= info["iters"] - 1:
            continue
        Y, i = la.inverse(A, max_iter=cap, raise_not_converged=False)
        torch.cuda.synchronize()
        assert i["iters"] == cap and i["stop_reason"] == 2
    with pytest.raises(la.LAError) as e:
        la.inverse(torch.full((n, m), float("nan"), device="cuda"))
    assert e.value.status == la.Status.NONFINITE
