"""Solves in one kernel (small sliced rows) against the three-kernel iteration:
the same operations in the same order of every sum, so x, the iteration count,
the status and the residual are the same bits -- over partial and misaligned
row ranges (1 row to the limits of 65 536 rows of one kernel form, 131 072 and
262 144 of the wide ones, and past them; odd vector chunks), line widths up to each register size and past the last, every way to stop, a
solve longer than one launch, new values, solves at the same time on two
streams (one of them then takes the launches), and a wait that gives up.
"""
import threading

import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.sym_expanded]
SOLVES = (dict(tol=1e-10, maxit=3000), dict(tol=1e-14, maxit=7), dict(tol=1e-3, maxit=0))


def both(monkeypatch, fmt, arrs, run):
    """run(solver) with the resident kernel and with three kernels."""
    out = []
    for fused in (None, "0"):
        if fused is None:
            monkeypatch.delenv("CGMI_FUSED", raising=False)
        else:
            monkeypatch.setenv("CGMI_FUSED", fused)
        with cgmi.Solver(fmt, *arrs) as S:
            out.append(run(S))
    monkeypatch.delenv("CGMI_FUSED", raising=False)
    return out


def solves(b, x0=None, opts=SOLVES):
    def run(S):
        res = []
        for o in opts:
            x, i = S.solve(to_dev(b), None if x0 is None else to_dev(x0), check=False, **o)
            res.append((x.cpu().numpy(), i["iters"], i["status"], i["relres"], i["relres_true"]))
        return res
    return run


def same(a, b, label):
    for r, q in zip(a, b):
        assert np.array_equal(r[0], q[0], equal_nan=True) and r[1:] == q[1:], (label, r[1:], q[1:])


def tridiagonal(n):
    i = np.arange(n)
    col = np.stack([i - 1, i, i + 1], axis=1)
    ok = (col >= 0) & (col < n)
    ptr = np.zeros(n + 1, np.int32)
    ptr[1:] = np.cumsum(ok.sum(axis=1))
    val = np.broadcast_to([-1.0, 2.5, -1.0], (n, 3))
    return ptr, col[ok].astype(np.int32), val[ok].copy()


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 300, 1000, 30001, 65535, 65536, 65537,
                               70001, 131072, 131073, 200000, 262144, 262145])
def test_row_ranges(monkeypatch, n):
    arrs = tridiagonal(n)
    say(f"resident tridiagonal n={n}")
    b, x0 = W.uniform_vector(n, seed=1), W.uniform_vector(n, seed=2)
    same(*both(monkeypatch, "csr", arrs, solves(b, x0)), n)


@pytest.mark.parametrize("per_row", [5, 9, 16, 24, 40])
def test_line_widths(monkeypatch, per_row):
    """Scattered columns (32-bit), so each row's columns are its own list."""
    n = 2000
    monkeypatch.setenv("CGMI_ROW_LAYOUT", "slices")
    arrs = W.random_spd_sparse(n, density=(per_row - 1) / n, seed=per_row)
    say(f"resident widths: longest row {np.diff(arrs[0]).max()}")
    same(*both(monkeypatch, "csr", arrs, solves(W.uniform_vector(n, seed=3))), per_row)


def test_wide_fem(monkeypatch):
    """The wide form on a grid whose product and vector rows do not align."""
    s = W.fem_p1_system(47, 45, 43, nu_iron=1e-2, seed=14)
    x0 = W.uniform_vector(s.n, seed=15)
    opts = (dict(tol=1e-8, maxit=3000), dict(tol=1e-14, maxit=1030))
    same(*both(monkeypatch, "csr", (s.rowptr, s.col, s.val), solves(s.b, x0, opts)), "wide")


@pytest.mark.parametrize("fmt", ["csr", "symcsr"])
def test_fem_and_stops(monkeypatch, fmt):
    s = W.fem_p1_system(21, 19, 17, nu_iron=1e-4, seed=4)
    arrs = (s.rowptr, s.col, s.val) if fmt == "csr" else W.upper_triangle(s.rowptr, s.col, s.val)
    opts = SOLVES + (dict(tol=1e-13, maxit=2500),)       # more iterations than one launch makes
    a, b = both(monkeypatch, fmt, arrs, solves(s.b, opts=opts))
    same(a, b, fmt)
    assert a[-1][1] > 1100, a[-1][1]
    nan, zero = s.b.copy(), np.zeros(s.n)
    nan[7] = np.nan
    x0 = W.uniform_vector(s.n, seed=5)
    for rhs in (nan, zero):
        same(*both(monkeypatch, fmt, arrs, solves(rhs, x0)), "b")


def test_breakdown(monkeypatch):
    n = 700
    d = np.where(np.arange(n) % 3 == 2, -1.0, 2.0)
    arrs = (np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), d)
    a, b = both(monkeypatch, "csr", arrs, solves(W.uniform_vector(n, seed=6)))
    same(a, b, "breakdown")
    assert a[0][2] == cgmi.CG_ERR_BREAKDOWN and a[0][1] > 0


def test_new_values(monkeypatch):
    s = W.fem_p1_system(13, 12, 11, seed=7)
    v = s.val * 3.0

    def run(S):
        first = solves(s.b)(S)
        S.set_values(to_dev(v))
        return first + solves(s.b)(S)
    same(*both(monkeypatch, "csr", (s.rowptr, s.col, s.val), run), "values")


def test_wait_gives_up(monkeypatch):
    """A wait that runs out at once: the solve is repeated with launches."""
    s = W.fem_p1_system(16, 15, 14, seed=8)
    arrs = (s.rowptr, s.col, s.val)
    x0 = W.uniform_vector(s.n, seed=9)
    with cgmi.Solver("csr", *arrs) as S:
        ref = solves(s.b, x0)(S)
    monkeypatch.setenv("CGMI_RESIDENT_WAIT", "-1")
    with cgmi.Solver("csr", *arrs) as S:
        same(ref, solves(s.b, x0)(S), "gives up")


def test_two_streams():
    """Two solves of 180 workgroups each cannot both be resident."""
    import torch
    s = W.fem_p1_system(36, 36, 35, seed=10)
    b = to_dev(s.b)
    with cgmi.Solver("csr", s.rowptr, s.col, s.val) as S:
        ref, info = S.solve(b)
    torch.cuda.synchronize()
    got = {}

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()), cgmi.Solver("csr", s.rowptr, s.col, s.val) as S:
            got[k] = [S.solve(b) for _ in range(5)]
            torch.cuda.current_stream().synchronize()
    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        for x, i in got[k]:
            assert torch.equal(x, ref) and i["iters"] == info["iters"]
