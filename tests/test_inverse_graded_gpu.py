"""la_inverse at AUTO of inputs whose entries differ widely in size: the polish step of an
uneven A or X runs at 6xBF16, so the result is the same bits as that of the workspace
without room for the fp16 polish; in between no column of X is worse than 1.25 times
that one's error, and 5e-7 (four FP32 units) for the draw."""
import ctypes

import pytest
import torch

import la_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def la():
    import paper_2112_09017_amd as la
    la.lib()
    return la


def run(la, A, short):
    n, m = A.shape
    o = la.make_inverse_opts()
    size = int(la.lib().la_inverse_workspace_size(n, m, ctypes.byref(o))) - short
    ws = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
    X = torch.empty((m, n), device="cuda")
    info = la.InverseInfo()
    st = la.lib().la_inverse(la.context(0), n, m, A.data_ptr(), m, X.data_ptr(), n,
                             (ws.data_ptr() + 255) & ~255, size, ctypes.byref(o),
                             ctypes.byref(info), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st == la.Status.OK
    return X, info.as_dict()


@pytest.mark.parametrize("kind", ["rows", "columns", "identity"])
@pytest.mark.parametrize("n,m", [(1800, 1800), (2300, 1800), (1800, 2300)])
@pytest.mark.parametrize("g", [2, 5])
def test_no_worse_than_x6(la, n, m, kind, g):
    r = min(n, m)
    A = torch.from_numpy(la_inputs.polar_case(max(n, m), r, 1.0, seeds=(61, 62, 63)).A32).cuda()
    A = (A if n >= m else A.T).contiguous()
    if kind == "rows":
        A = A * 2.0 ** -torch.linspace(0, g, n, device="cuda")[:, None]
    elif kind == "columns":
        A = A * 2.0 ** -torch.linspace(0, g, m, device="cuda")[None, :]
    else:      # 1 on the diagonal, 2^-4g elsewhere
        A = torch.eye(n, m, device="cuda") + 2.0 ** (-4 * g) * A
    A = A.contiguous()
    (X, i0), (Y, i1) = run(la, A, 0), run(la, A, 1)
    assert i0["iters"] == i1["iters"]
    want = torch.linalg.pinv(A.double().cpu()).cuda() if n != m else torch.linalg.inv(A.double())
    if kind == "identity":
        off = ~torch.eye(m, n, dtype=torch.bool, device="cuda")
        e = [(torch.linalg.norm((Z.double() - want)[off]) / torch.linalg.norm(want[off])).item()
             for Z in (X, Y)]
        if g == 5:
            assert torch.equal(X, Y)
    else:
        e = [(torch.linalg.norm(Z.double() - want, dim=0) / torch.linalg.norm(want, dim=0)).max().item()
             for Z in (X, Y)]
    print(kind, n, m, g, e)
    assert e[0] <= 1.25 * e[1] + 5e-7


def test_even_inputs_take_the_fp16_terms(la):
    A = torch.from_numpy(la_inputs.polar_case(1800, 1800, 0.1, seeds=(61, 62, 63)).A32).cuda()
    assert not torch.equal(run(la, A, 0)[0], run(la, A, 1)[0])


@pytest.mark.parametrize("cond", [200.0])
def test_more_steps_than_the_first_batch(la, cond):
    """Steps are queued 16 at a time at first: an input that needs more, and the caps around
    the border of the batch."""
    A = torch.from_numpy(la_inputs.polar_case(400, 400, 1.0 / cond, seeds=(64, 65, 66)).A32).cuda()
    X, info = la.inverse(A)
    assert info["stop_reason"] == 0 and info["iters"] > 18
    R = X.double() @ A.double() - torch.eye(400, dtype=torch.float64, device="cuda")
    assert torch.linalg.norm(R).item() / 20.0 <= 2e-6 * cond ** 2
    for cap in (15, 16, 17):
        Y, i = la.inverse(A, max_iter=cap, raise_not_converged=False)
        Z, j = la.inverse(A, max_iter=cap - 1, raise_not_converged=False)
        torch.cuda.synchronize()
        assert i["iters"] == cap and i["stop_reason"] == 2 and j["iters"] == cap - 1
        want = torch.linalg.norm(Y.double() - Z.double()).item() * i["gram_norm"] ** 0.5
        assert abs(i["last_delta"] - want) <= 1e-6 * want
