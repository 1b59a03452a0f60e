"""The layout by rows beside CSC panels and compact symmetric blocks: products
and solves then have the bits of the same matrix given as CSR -- new values,
lower triangles, non-symmetric and ragged columns (empty ones; too ragged for
slices: the panels), sizes on both sides of the one that a solve changes at."""
import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import check_spmv, say, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.sym_expanded]


@pytest.mark.parametrize("kind", ["csc_small", "csc", "symcsr", "lower"])
def test_rows_have_csr_bits(kind):
    s = W.fem_p1_system(*((13, 12, 11) if kind == "csc_small" else (43, 42, 40)), nu_iron=0.5, seed=1)
    base = (s.rowptr, s.col, s.val)
    fmt, arrs, flags, scale = "csc", base, 0, np.arange(s.nnz) * 0.0 + 1.5
    if kind in ("symcsr", "lower"):
        fmt, arrs = "symcsr", W.upper_triangle(*base)
        if kind == "lower":
            arrs, flags = W.transpose_csr(s.n, s.n, *arrs), cgmi.CG_LOWER
    say(f"rows {kind} n={s.n}")
    x, x0 = to_dev(W.uniform_vector(s.n, seed=2)), to_dev(W.uniform_vector(s.n, seed=3))
    out = []
    for f, a, fl in (("csr", base, 0), (fmt, arrs, flags)):
        with cgmi.Solver(f, *a, flags=fl) as S:
            res = [S.spmv(x), S.spmv_static(x)]
            for kw in (dict(tol=1e-9, maxit=2000), dict(x0=x0, tol=1e-14, maxit=11)):
                res += [S.solve(to_dev(s.b), **kw)[0]]
            S.set_values(to_dev(a[2] * 1.5))
            res += [S.spmv(x), S.solve(to_dev(s.b), tol=1e-9, maxit=2000)[0]]
            out.append([r.cpu().numpy() for r in res])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("kind", ["banded", "ragged"])
def test_csc_products(kind):
    if kind == "banded":
        ptr, idx, val = W.banded_sparse(9000, 40, density=0.2, seed=4, empty=50)
    else:
        ptr, idx, val = W.random_sparse(900, density=0.02, seed=5, empty_rows=60, long_rows=4, long_len=800)
    x = W.uniform_vector(len(ptr) - 1, seed=6)
    check_spmv(cgmi.CG_FMT_CSC, ptr, idx, val, x, label=f"rows {kind}")
    check_spmv(cgmi.CG_FMT_CSC, ptr + 1, idx + 1, val, x, base=1, label=f"rows {kind} 1-based")
