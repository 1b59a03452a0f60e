"""CSC handles that hold both layouts: products by rows, solves (past 262 144
rows) and refinements (CG_MIXED) on the panels.  After new values, which reach
the rows from the caller's order or through the panels' slots, both layouts have
the bits of a handle made with those values; products follow the oracle, and
solves the CSR handle's solution.
"""
import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import check_spmv, say, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.sym_expanded]


@pytest.fixture(params=["0", "1"], ids=["values from the caller", "values through the panels"])
def way(request, monkeypatch):
    monkeypatch.setenv("CGMI_ROWS_FROM_PANELS", request.param)


def nonsymmetric(n, seed):
    """Columns with rows j - 5, j, j + 3 and j + 1900, 500 of them empty."""
    j = np.delete(np.arange(n), np.arange(n // 3, n // 3 + 500))
    i = j[:, None] + np.array([-5, 0, 3, 1900])
    ok = (i >= 0) & (i < n)
    ptr = np.zeros(n + 1, np.int64)
    ptr[j + 1] = ok.sum(axis=1)
    return np.cumsum(ptr).astype(np.int32), i[ok].astype(np.int32), W.uniform_vector(int(ok.sum()), seed=seed)


@pytest.mark.parametrize("n", [262145, 262209, 300000])
def test_products_after_new_values(n, way):
    """Empty columns, partial last slices and panels, a matrix that is not symmetric."""
    ptr, idx, val = nonsymmetric(n, n % 97)
    x = W.uniform_vector(n, seed=1)
    new = W.uniform_vector(len(idx), seed=2)
    with cgmi.Solver("csc", ptr, idx, val) as S, cgmi.Solver("csc", ptr, idx, new) as F:
        st = S.stats()
        say(f"beside n={n}: {st}")
        assert st["slots"] > 0 and st["slices"] == 2  # (panels as well as rows)
        check_spmv(cgmi.CG_FMT_CSC, ptr, idx, val, x, solver=S, label="old values")
        S.set_values(to_dev(new))
        y, _ = check_spmv(cgmi.CG_FMT_CSC, ptr, idx, new, x, solver=S, label="new values")
        assert np.array_equal(y, F.spmv(to_dev(x)).cpu().numpy())
        assert np.array_equal(y, S.spmv_static(to_dev(x)).cpu().numpy())


@pytest.mark.parametrize("grid", [(64, 64, 64), (65, 64, 64)])
def test_solves_on_both_sides_of_the_limit(grid, way):
    """262 144 rows are solved by rows (the bits of CSR), 266 240 on the panels."""
    s = W.fem_p1_system(*grid, nu_iron=0.5, seed=3)
    b = to_dev(s.b)
    new = to_dev(s.val * 1.5)
    out = {}
    for fmt in ("csr", "csc"):
        with cgmi.Solver(fmt, s.rowptr, s.col, s.val) as S, cgmi.Solver(fmt, s.rowptr, s.col, s.val * 1.5) as F:
            res = [S.solve(b, tol=1e-9)]
            S.set_values(new)
            res += [S.solve(b, tol=1e-9), F.solve(b, tol=1e-9)]
            path = S.report()["path"]
            assert np.array_equal(res[1][0].cpu().numpy(), res[2][0].cpu().numpy())
            assert path == (cgmi.CG_PATH_RESIDENT if s.n <= 262144 else cgmi.CG_PATH_LAUNCHES)
            out[fmt] = [(r[0].cpu().numpy(), r[1]["iters"]) for r in res]
    for (xr, ir), (xc, ic) in zip(out["csr"], out["csc"]):
        if s.n <= 262144:
            assert np.array_equal(xr, xc) and ir == ic
        else:  # (another order of every sum: two solutions to 1e-9 of their residuals)
            assert np.linalg.norm(xr - xc) <= 1e-6 * np.linalg.norm(xr)


@pytest.mark.parametrize("fmt", ["csc", "symcsr", "lower"])
def test_mixed_with_rows(fmt, way):
    """cg_solve resident by rows, cg_solve_mixed on the format's own layout."""
    s = W.fem_p1_system(43, 42, 40, nu_iron=0.5, seed=4)
    full, flags, kind = (s.rowptr, s.col, s.val), 0, fmt
    arrs = full
    if fmt != "csc":
        arrs, kind = W.upper_triangle(*full), "symcsr"
        if fmt == "lower":
            arrs, flags = W.transpose_csr(s.n, s.n, *arrs), cgmi.CG_LOWER
    b, v = to_dev(s.b), arrs[2] * 1.5
    with cgmi.Solver(kind, *arrs, flags=flags, mixed=True) as S, \
            cgmi.Solver(kind, arrs[0], arrs[1], v, flags=flags, mixed=True) as F, \
            cgmi.Solver("csr", s.rowptr, s.col, s.val * 1.5) as R:
        S.set_values(to_dev(v))
        x = S.solve(b, tol=1e-10)[0].cpu().numpy()
        assert S.report()["path"] == cgmi.CG_PATH_RESIDENT
        assert np.array_equal(x, R.solve(b, tol=1e-10)[0].cpu().numpy())
        assert np.array_equal(S.spmv(b).cpu().numpy(), R.spmv(b).cpu().numpy())
        m, info = S.solve_mixed(b, tol=1e-11)
        assert S.report()["path"] == cgmi.CG_PATH_LAUNCHES and info["status"] == cgmi.CG_OK
        assert np.array_equal(m.cpu().numpy(), F.solve_mixed(b, tol=1e-11)[0].cpu().numpy())
        assert np.linalg.norm(m.cpu().numpy() - x) <= 1e-6 * np.linalg.norm(x)


@pytest.mark.parametrize("fmt", ["csc", "symcsr"])
def test_values_that_mixed_precision_refuses(fmt, way):
    """A diagonal entry that is not positive: the call says so, and the FP64
    matrix has its new values in every layout all the same."""
    s = W.fem_p1_system(43, 42, 40, nu_iron=0.5, seed=5)
    full = (s.rowptr, s.col, s.val)
    ptr, col, val = W.upper_triangle(*full) if fmt == "symcsr" else full
    new = val * 1.5
    line = np.repeat(np.arange(s.n), np.diff(ptr))
    new[np.nonzero((line == col) & (line == s.n // 2))[0][0]] = -1.0
    x = to_dev(W.uniform_vector(s.n, seed=6))
    with cgmi.Solver(fmt, ptr, col, val, mixed=True) as S, cgmi.Solver(fmt, ptr, col, new) as F:
        with pytest.raises(cgmi.CgError) as e:
            S.set_values(to_dev(new))
        assert e.value.status == cgmi.CG_ERR_ARG
        assert np.array_equal(S.spmv(x).cpu().numpy(), F.spmv(x).cpu().numpy())
        S.set_values(to_dev(val))
        assert S.solve_mixed(to_dev(s.b), tol=1e-10)[1]["status"] == cgmi.CG_OK
