"""The inverse's polish step at AUTO on scaled fp16 terms.

Against the exact inverse in FP64 the result is no worse than that of the same steps
polished at 6xBF16 (the workspace without the region that the fp16 polish needs):
its products round half as often, so 1.05 covers the draw.  Rows and columns
scaled apart by powers of two leave the same digits in the operands."""
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
    return X.double()


@pytest.mark.parametrize("n,m", [(1700, 1700), (2049, 2049), (1800, 2300), (2300, 1800)])
def test_polish_error(la, n, m):
    r = min(n, m)
    case = la_inputs.polar_case(max(n, m), r, 1.0 / 20.0, seeds=(61, 62, 63))
    A = torch.from_numpy(case.A32).cuda()
    A = (A if n >= m else A.T).contiguous()
    want = torch.linalg.pinv(A.double().cpu()).cuda()
    e = [(torch.linalg.norm(run(la, A, s) - want) / torch.linalg.norm(want)).item()
         for s in (0, 1)]
    print(f"\n{n} x {m}: fp16 {e[0]:.3g}, 6xBF16 {e[1]:.3g}")
    assert e[0] <= 1.05 * e[1]
