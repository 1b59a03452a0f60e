"""New values and value gradients of a planned matrix, at the edges of the
kernels that move them: 64-line groups (1, 63, 64, 65, 130 lines), runs longer
than the staged 1024 entries of a slice or the 1024-entry map of a gradient
window, empty lines, odd and even widths, every format and layout.  Both are
exact: the product after cg_set_values has the bits of a handle made with those
values, a gradient the bits of its rounded products.
"""
import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def matrices():
    for n in (1, 63, 64, 65, 130):
        s = W.random_spd_sparse(n, density=0.05, seed=n)
        yield f"spd{n}", s
    yield "wide", W.random_spd_sparse(200, density=0.5, seed=5)       # ~100 a row: 6400 in 64 lines
    s = W.fem_p1_system(17, 9, 13, seed=6, with_rhs=False)
    yield "fem", (s.rowptr, s.col, s.val)
    yield "ragged", W.random_sparse(300, density=0.02, seed=7, empty_rows=20, long_rows=2, long_len=280)


@pytest.mark.parametrize("layout", ["", "slices", "rows"])
@pytest.mark.parametrize("fmt", ["csr", "symcsr", "lower", "csc"])
def test_values_and_gradients_exact(fmt, layout, monkeypatch):
    if layout:
        monkeypatch.setenv("CGMI_ROW_LAYOUT", layout)
    for name, (ptr, col, val) in matrices():
        if fmt in ("symcsr", "lower") and name == "ragged":
            continue
        n, flags = len(ptr) - 1, 0
        if fmt == "symcsr":
            ptr, col, val = W.upper_triangle(ptr, col, val)
        elif fmt == "lower":
            up = W.upper_triangle(ptr, col, val)
            ptr, col, val = W.transpose_csr(n, n, *up)
            flags = cgmi.CG_LOWER
        say(f"{fmt} {layout} {name} n={n} nnz={len(col)}")
        kind = "symcsr" if fmt == "lower" else fmt
        rng = np.random.default_rng(8)
        new, lam, x = (rng.uniform(-1, 1, size=k) for k in (len(col), n, n))
        with cgmi.Solver(kind, ptr, col, val, flags=flags) as S, cgmi.Solver(kind, ptr, col, new, flags=flags) as F:
            S.set_values(to_dev(new))
            assert np.array_equal(S.spmv(to_dev(x)).cpu().numpy(), F.spmv(to_dev(x)).cpu().numpy()), name
            g = S.pattern_grad(to_dev(lam), to_dev(x)).cpu().numpy()
        line = np.repeat(np.arange(n), np.diff(ptr))
        if fmt == "csr":
            ref = -(lam[line] * x[col])
        elif fmt == "csc":
            ref = -(lam[col] * x[line])
        else:
            i, j = np.minimum(line, col), np.maximum(line, col)  # the upper entry's row and column
            ref = np.where(i == j, -(lam[i] * x[j]), -(lam[i] * x[j] + lam[j] * x[i]))
        assert np.array_equal(g, ref), name
