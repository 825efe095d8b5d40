"""Polar iterations whose products hand their results on as packed operands.

la_polar with the workspace its size function asks for runs the steps of small
sizes on packed operands, one a byte shorter on FP32 operands; the server does
so for requests that are small beside its arena.  The operand terms, the order of
every sum and of the step norm's partial sums are the same, so U, H and the info
agree bit for bit.  The workspace is filled with NaN bytes first: no product may
use what the products before it did not write."""
import ctypes
import time

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


def run(la, A, short, ldu_pad, opts):
    m, n = A.shape
    o = la.make_opts(**opts)
    size = int(la.lib().la_polar_workspace_size(m, n, ctypes.byref(o)))
    ws = torch.full((size + 256,), 255, dtype=torch.uint8, device="cuda")
    U = torch.full((m, n + ldu_pad), 7.0, device="cuda")
    H = torch.empty((n, n), device="cuda")
    info = la.PolarInfo()
    p = (ws.data_ptr() + 255) & ~255
    st = la.lib().la_polar(la.context(0), m, n, A.data_ptr(), A.stride(0), U.data_ptr(),
                           n + ldu_pad, H.data_ptr(), n, p, size - short, ctypes.byref(o),
                           ctypes.byref(info), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    if st != la.Status.OK:
        return st
    assert torch.all(U[:, n:] == 7.0)
    return U[:, :n].clone(), H, info.as_dict()


SHAPES = [(5, 3), (33, 17), (64, 64), (65, 63), (129, 127), (257, 193), (320, 320), (400, 321), (512, 511),
          (640, 256), (641, 641), (700, 641), (1001, 1001), (1500, 1025)]
OPTS = {"default": {}, "x3": dict(prec_precond=2, prec_ns=2), "no_precond": dict(s0=0.5),
        "polish": dict(polish=True)}


@pytest.mark.parametrize("opts", list(OPTS))
@pytest.mark.parametrize("shape", SHAPES)
def test_chained_equals_plain(la, shape, opts):
    m, n = shape
    s_min = 0.6 if opts == "no_precond" else 1e-2
    A = torch.from_numpy(la_inputs.polar_case(m, n, s_min, seeds=(71 + m, 72 + n, 73)).A32).cuda()
    for pad in (0, 5):
        full = run(la, A, 0, pad, OPTS[opts])
        short = run(la, A, 1, pad, OPTS[opts])
        if n < 320:   # no packed copies to leave out
            assert short == la.Status.OUT_OF_MEMORY
            continue
        assert torch.equal(full[0], short[0]) and torch.equal(full[1], short[1])
        assert full[2] == short[2]
        assert torch.isfinite(full[0]).all()


def test_server_chained_equals_plain(la):
    cs = [la_inputs.polar_case(m, n, 1e-2, seeds=(81 + m, 82 + n, 83)).A32
          for m, n in [(130, 97), (333, 333), (700, 641), (1001, 1001)]]
    out = []
    for arena in (1 << 30, 100 << 20):
        with la.Server(arena, max_slots=8) as srv:
            ids = [srv.submit(a) for a in cs for _ in range(2)]
            got, t0 = {}, time.time()
            while len(got) < len(ids) and time.time() - t0 < 60:
                for i in ids:
                    r = None if i in got else srv.poll(i)
                    if r is not None:
                        got[i] = r
                time.sleep(0.001)
            out.append([got[i] for i in ids])
    for a, b in zip(*out):
        assert a[0] == b[0] == la.Status.OK
        assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2]) and a[3] == b[3]


@pytest.mark.parametrize("opts", [{}, dict(polish=True), dict(prec_precond=3, prec_ns=3),
                                  dict(prec_precond=1, prec_ns=1)],
                         ids=["default", "polish", "x6", "fp32"])
def test_server_equals_polar(la, opts):
    """One launch per phase takes every request in flight, whatever its size and
    arithmetic: each tile is the sums of la_polar's launch in their order (below
    4096 rows neither splits K), so the factors agree bit for bit."""
    cs = [la_inputs.polar_case(m, n, 1e-2, seeds=(91 + m, 92 + n, 93)).A32
          for m, n in [(1, 1), (40, 31), (130, 97), (300, 257), (700, 641), (1001, 1001)]]
    with la.Server(1 << 30, max_slots=8) as srv:
        ids = [srv.submit(a, **opts) for a in cs]
        got, t0 = {}, time.time()
        while len(got) < len(ids) and time.time() - t0 < 60:
            for i in ids:
                r = None if i in got else srv.poll(i)
                if r is not None:
                    got[i] = r
            time.sleep(0.001)
    for a, i in zip(cs, ids):
        U, H, info = la.polar(torch.from_numpy(a).cuda(), **opts)
        st, U2, H2, info2 = got[i]
        assert st == la.Status.OK
        assert np.array_equal(U.cpu().numpy(), U2) and np.array_equal(H.cpu().numpy(), H2)
        assert info["iters_ns"] == info2["iters_ns"]
