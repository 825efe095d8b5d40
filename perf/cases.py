"""Timed workloads of the library: its public calls over the sizes users bring.

``listed()`` names twelve cases, from a 256^3 product to the 16384^2 polar
factorisation; ``draw(rng)`` gives further cases of the same ranges.
``prepare`` makes the inputs and the workspaces, outputs and servers a calling
program keeps, ``run`` makes one pass through the public entry points and
returns everything it computed, ``exact`` gives the same results from plain
FP64 torch, and ``work`` the bytes and operations a pass cannot do without.

Polar and inverse inputs are A = Q diag(s) V^T with s_1 = 1, s_n = 1/cond and
the rest log-uniform between, Q and V random orthogonal.  Their condition
numbers are 10 to 30, the lower end of the serving mix, where the factors
themselves (and not just the residual) are determined to FP32 accuracy.
Products and QR take i.i.d. N(0, 1) entries.
"""
from __future__ import annotations

import math
import time

import torch

import paper_2112_09017_amd as la

DEV = "cuda:0"


# ------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest product: one launch, its latency is all that counts
        {"name": "gemm_256", "op": "gemm", "m": 256, "n": 256, "k": 256, "ta": False,
         "tb": False, "prec": "BF16X3", "alpha": 1.0},
        # an ordinary product of odd sizes with a transposed operand, at FP32-level accuracy
        {"name": "gemm_ragged_x6", "op": "gemm", "m": 1500, "n": 1101, "k": 2300, "ta": True,
         "tb": False, "prec": "BF16X6", "alpha": 0.5},
        # the paper's per-core block product (the benchmark's headline), workspace kept
        {"name": "gemm_block", "op": "gemm_ws", "m": 16384, "n": 16384, "k": 32768,
         "ta": False, "tb": False, "prec": "BF16X3", "alpha": 1.0},
        # the smallest polar of the repository's configurations: launches and read-backs
        {"name": "polar_256", "op": "polar", "m": 256, "n": 256, "cond": 30.0},
        # a mid-size polar that is a multiple of no tile
        {"name": "polar_1000", "op": "polar", "m": 1000, "n": 1000, "cond": 20.0},
        # the benchmark's square polar
        {"name": "polar_16384", "op": "polar", "m": 16384, "n": 16384, "cond": 30.0},
        # the benchmark's tall polar (orthogonalising many vectors)
        {"name": "polar_tall", "op": "polar", "m": 131072, "n": 4096, "cond": 10.0},
        # inversion of an ordinary odd-sized matrix
        {"name": "inverse_3000", "op": "inverse", "n": 3000, "m": 3000, "cond": 20.0},
        # a function of a symmetric matrix, degree 16 as in the benchmark
        {"name": "cheb_4096", "op": "cheb", "n": 4096, "degree": 16},
        # the benchmark's tall QR panel (Gram-Schmidt of 64 vectors)
        {"name": "tsqr_131072x64", "op": "tsqr", "m": 131072, "n": 64},
        # QR with Q of a least-squares matrix
        {"name": "caqr_6144x4096", "op": "caqr", "m": 6144, "n": 4096, "panel": 64,
         "want_q": True},
        # a burst of mixed requests to the polar server, host arrays in and out
        {"name": "serve_mix", "op": "serve", "count": 12, "lo": 128, "hi": 1536, "order": 1},
    ]


def _log_int(rng, lo, hi):
    """An integer log-uniform in [lo, hi]; half of them odd as drawn, half multiples of 64."""
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5 and x >= 64:
        x = 64 * max(1, round(x / 64))
    return max(lo, min(hi, x))


def draw(rng):
    op = rng.choice(["gemm", "gemm", "gemm_ws", "polar", "polar", "inverse", "cheb", "odd", "tsqr",
                     "caqr", "serve"])
    if op == "gemm":
        return {"op": op, "m": _log_int(rng, 64, 8192), "n": _log_int(rng, 64, 8192),
                "k": _log_int(rng, 64, 8192), "ta": rng.random() < 0.5, "tb": rng.random() < 0.5,
                "prec": rng.choice(["BF16X3", "BF16X6", "FP32"]),
                "alpha": rng.choice([1.0, 0.5, -1.0])}
    if op == "gemm_ws":
        return {"op": op, "m": _log_int(rng, 2048, 16384), "n": _log_int(rng, 2048, 16384),
                "k": _log_int(rng, 1024, 16384), "ta": rng.random() < 0.5,
                "tb": rng.random() < 0.5, "prec": "BF16X3", "alpha": 1.0}
    if op == "polar":
        n = _log_int(rng, 128, 6144)
        m = n if rng.random() < 0.5 else _log_int(rng, n, 8 * n)
        return {"op": op, "m": m, "n": n, "cond": round(10.0 ** rng.uniform(1.0, 1.5), 2)}
    if op == "inverse":
        n = _log_int(rng, 128, 6144)
        m = n if rng.random() < 0.7 else _log_int(rng, n // 4, n)
        if rng.random() < 0.5:
            n, m = m, n
        return {"op": op, "n": n, "m": m, "cond": round(10.0 ** rng.uniform(1.0, 1.5), 2)}
    if op == "cheb":
        return {"op": op, "n": _log_int(rng, 128, 6144), "degree": rng.randint(4, 24)}
    if op == "odd":
        n = _log_int(rng, 128, 6144)
        return {"op": op, "m": _log_int(rng, max(96, n // 2), 3 * n), "n": n,
                "terms": rng.randint(2, 8)}
    if op == "tsqr":
        n = rng.randint(4, 128)
        return {"op": op, "m": _log_int(rng, 1024, 262144), "n": n}
    if op == "caqr":
        n = _log_int(rng, 128, 4096)
        return {"op": op, "m": int(n * rng.uniform(1.25, 4.0)), "n": n,
                "panel": rng.choice([32, 64, 64, 128]), "want_q": rng.random() < 0.5}
    return {"op": op, "count": rng.randint(2, 16), "lo": 128, "hi": rng.choice([512, 1024, 2048]),
            "order": rng.randint(2, 1 << 20)}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _gauss(shape, g):
    return torch.randn(shape, generator=g, dtype=torch.float32, device=DEV)


def _signs(n, g):
    return (2 * torch.randint(0, 2, (n,), generator=g, device=DEV) - 1).to(torch.float32)


def _hartley(m, n, g):
    """n columns of the m x m Hartley matrix cas(2 pi j k / m) / sqrt(m), rows
    in random order with random signs: orthonormal columns for any m."""
    rows = torch.randperm(m, generator=g, device=DEV)
    out = torch.empty((m, n), dtype=torch.float32, device=DEV)
    k = torch.arange(n, device=DEV)
    w = _signs(m, g) / math.sqrt(m)
    for r in range(0, m, 8192):
        x = ((rows[r:r + 8192, None] * k[None, :]) % m).to(torch.float64) * (2.0 * math.pi / m)
        out[r:r + 8192] = (torch.cos(x) + torch.sin(x)).to(torch.float32) * w[r:r + 8192, None]
        del x
    return out


def _with_spectrum(m, n, cond, g):
    """m x n (m >= n) A = Q diag(s) V^T, s_1 = 1, s_n = 1/cond, log-uniform between."""
    s = torch.exp(torch.rand(n, generator=g, dtype=torch.float64, device=DEV) * -math.log(cond))
    s[0] = 1.0
    s[-1] = 1.0 / cond
    q = _hartley(m, n, g)
    q *= (_signs(n, g).double() * s).to(torch.float32)[None, :]
    return q @ _hartley(n, n, g).t()


def _symmetric(n, g):
    a = _gauss((n, n), g)
    return ((a + a.t()) * (0.25 / math.sqrt(n))).contiguous()


def _cheb_coef(degree):
    """Chebyshev coefficients of exp(-x) to the given degree (modified Bessel values, by series)."""
    def bessel_i(k):
        return sum(0.5 ** (2 * j + k) / (math.factorial(j) * math.factorial(j + k))
                   for j in range(24))
    return [(1 if k == 0 else 2) * (-1) ** k * bessel_i(k) for k in range(degree + 1)]


def _odd_coef(terms):
    """Alternating, slowly falling coefficients of x, x^3, x^5, ..."""
    return [(-1) ** j * 0.9 / (j + 1) for j in range(terms)]


def _serve_shapes(case):
    """Square sizes log-uniform in [lo, hi], in the order the case's own number gives."""
    import random
    r = random.Random(case["order"])
    return [_log_int(r, case["lo"], case["hi"]) for _ in range(case["count"])]


def _serve_inputs(case, seed):
    g = _gen(seed)
    return [_with_spectrum(n, n, 10.0 + 20.0 * i / case["count"], g)
            for i, n in enumerate(_serve_shapes(case))]


def _inputs(case, seed):
    g = _gen(seed)
    op = case["op"]
    if op in ("gemm", "gemm_ws"):
        a = _gauss((case["k"], case["m"]) if case["ta"] else (case["m"], case["k"]), g)
        b = _gauss((case["n"], case["k"]) if case["tb"] else (case["k"], case["n"]), g)
        return a.t() if case["ta"] else a, b.t() if case["tb"] else b
    if op == "polar":
        return _with_spectrum(case["m"], case["n"], case["cond"], g)
    if op == "inverse":
        n, m = case["n"], case["m"]
        a = _with_spectrum(max(n, m), min(n, m), case["cond"], g)
        return a if n >= m else a.t().contiguous()
    if op == "cheb":
        return _symmetric(case["n"], g)
    if op == "odd":
        return _gauss((case["m"], case["n"]), g) / (math.sqrt(case["m"]) + math.sqrt(case["n"]))
    return _gauss((case["m"], case["n"]), g)     # tsqr, caqr


def _bytes(n):
    return torch.empty(n + 256, dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    op = case["op"]
    st = {"case": case}
    if op == "serve":
        st["A"] = [a.cpu().numpy() for a in _serve_inputs(case, seed)]
        st["server"] = la.Server(3 << 30, max_slots=32)
        return st
    x = _inputs(case, seed)
    if op in ("gemm", "gemm_ws"):
        st["A"], st["B"] = x
        st["C"] = torch.empty((case["m"], case["n"]), dtype=torch.float32, device=DEV)
        st["prec"] = la.Precision[case["prec"]]
        if op == "gemm_ws":
            st["ws"] = _bytes(la.gemm_workspace_size(case["m"], case["n"], case["k"]))
        return st
    st["A"] = x
    if op == "polar":
        m, n = x.shape
        st["U"] = torch.empty_like(x)
        st["H"] = torch.empty((n, n), dtype=torch.float32, device=DEV)
        st["ws"] = _bytes(la.polar_workspace_size(m, n))
    elif op == "inverse":
        st["X"] = torch.empty((x.shape[1], x.shape[0]), dtype=torch.float32, device=DEV)
        st["ws"] = _bytes(la.inverse_workspace_size(x.shape[0], x.shape[1]))
    elif op in ("cheb", "odd"):
        st["F"] = torch.empty_like(x)
        st["ws"] = _bytes(la.lib().la_matfunc_workspace_size(x.shape[0], x.shape[1]))
    elif op == "caqr":
        st["ws"] = _bytes(la.caqr_workspace_size(x.shape[0], x.shape[1], case["panel"],
                                                 case["want_q"]))
    return st


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "gemm":
        return la.gemm(st["A"], st["B"], st["C"], alpha=case["alpha"], prec=st["prec"])
    if op == "gemm_ws":
        return la.gemm_ws(st["A"], st["B"], st["C"], alpha=case["alpha"], prec=st["prec"],
                          workspace=st["ws"])
    if op == "polar":
        u, h, _ = la.polar(st["A"], U=st["U"], H=st["H"], workspace=st["ws"])
        return {"U": u, "H": h}
    if op == "inverse":
        return la.inverse(st["A"], X=st["X"], workspace=st["ws"])[0]
    if op == "cheb":
        return la.matfunc_cheb(st["A"], -1.25, 1.25, _cheb_coef(case["degree"]), F=st["F"],
                               workspace=st["ws"])
    if op == "odd":
        return la.matfunc_odd(st["A"], _odd_coef(case["terms"]), F=st["F"], workspace=st["ws"])
    if op == "tsqr":
        q, r = la.tsqr(st["A"])
        return {"Q": q, "R": r}
    if op == "caqr":
        q, r = la.caqr(st["A"], panel=case["panel"], want_q=case["want_q"], workspace=st["ws"])
        return {"Q": q, "R": r} if case["want_q"] else {"R": r}
    srv = st["server"]
    ids = [srv.submit(a) for a in st["A"]]
    out = [None] * len(ids)
    left = set(range(len(ids)))
    while left:
        for i in sorted(left):
            r = srv.poll(ids[i])
            if r is not None:
                if r[0] != la.Status.OK:
                    raise RuntimeError(f"request {i} ended with {r[0]}")
                out[i] = {"U": r[1], "H": r[2]}
                left.discard(i)
        time.sleep(0.0001)
    return out


# ------------------------------------------------------------------- FP64

def _polar64(a):
    """U and H of A in FP64, by Newton-Schulz from A / ||A||_2 (estimated)."""
    a = a.double()
    n = a.shape[1]
    v = torch.ones((n, 1), dtype=torch.float64, device=a.device) / math.sqrt(n)
    v += 0.1 * torch.randn((n, 1), generator=_gen(1), dtype=torch.float64, device=a.device)
    for _ in range(20):
        v = a.t() @ (a @ v)
        v /= torch.linalg.norm(v)
    u = a / (1.1 * torch.linalg.norm(a @ v))
    for _ in range(60):
        g = u.t() @ u
        g.mul_(-0.5)
        g.diagonal().add_(1.5)
        new = u @ g
        done = float(torch.linalg.norm(new - u)) < 1e-9 * math.sqrt(n)
        u = new
        if done:
            break
    h = u.t() @ a
    return {"U": u, "H": 0.5 * (h + h.t())}


def exact(case, seed):
    op = case["op"]
    if op in ("tsqr", "caqr"):
        return None        # Q and R are unique only up to the signs the tree gives
    if op == "serve":
        return [_polar64(a) for a in _serve_inputs(case, seed)]
    x = _inputs(case, seed)
    if op in ("gemm", "gemm_ws"):
        return case["alpha"] * (x[0].double() @ x[1].double())
    if op == "polar":
        return _polar64(x)
    a = x.double()
    n, m = a.shape
    if op == "inverse":
        if n == m:
            return torch.linalg.inv(a)
        if n > m:
            return torch.linalg.solve(a.t() @ a, a.t().contiguous())
        return torch.linalg.solve(a @ a.t(), a).t().contiguous()
    if op == "odd":
        c = _odd_coef(case["terms"])
        g = a.t() @ a
        p = torch.zeros_like(g)
        for cj in reversed(c):
            p = p @ g
            p.diagonal().add_(cj)
        return a @ p
    c = _cheb_coef(case["degree"])
    b = a / 1.25
    t0 = torch.eye(n, dtype=torch.float64, device=a.device)
    t1 = b
    f = c[0] * t0 + c[1] * t1
    for ck in c[2:]:
        t0, t1 = t1, 2.0 * (b @ t1) - t0
        f += ck * t1
    return f


# ------------------------------------------------------------------- work

def _polar_work(m, n):
    # 15 preconditioning and about 9 Newton-Schulz steps, each a symmetric Gram (m n^2) and
    # an update (2 m n^2), then H (2 m n^2); A in, U and H out
    return 4.0 * (2 * m * n + n * n), (3 * 24 + 2) * float(m) * n * n


def work(case):
    op = case["op"]
    if op in ("gemm", "gemm_ws"):
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 4.0 * (m * k + k * n + m * n), "flops": 2.0 * m * n * k}
    if op == "polar":
        b, f = _polar_work(case["m"], case["n"])
    elif op == "inverse":
        # about 20 steps of two products, and the starting Gram norm (symmetric)
        n, m = case["n"], case["m"]
        small = min(n, m)
        b, f = 8.0 * n * m, (4 * 20 + 1) * float(n) * m * small
    elif op == "cheb":
        n = case["n"]
        b, f = 8.0 * n * n, 2.0 * (case["degree"] - 1) * float(n) ** 3
    elif op == "odd":
        m, n = case["m"], case["n"]
        b = 8.0 * m * n
        f = 3.0 * m * n * n + 2.0 * (case["terms"] - 2) * float(n) ** 3
    elif op == "tsqr":
        m, n = case["m"], case["n"]
        b, f = 4.0 * (2 * m * n + n * n), 4.0 * m * n * n - 4.0 / 3.0 * float(n) ** 3
    elif op == "caqr":
        m, n = case["m"], case["n"]
        q = 2 if case["want_q"] else 1
        b = 4.0 * (m * n * q + n * n)
        f = q * (2.0 * m * n * n - 2.0 / 3.0 * float(n) ** 3)
    else:
        parts = [_polar_work(n, n) for n in _serve_shapes(case)]
        b, f = sum(p[0] for p in parts), sum(p[1] for p in parts)
    return {"bytes": b, "flops": f}
