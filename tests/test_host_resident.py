"""The plan of a resident solve, checked on the CPU against the matrix: the
column list of each workgroup is the ascending set of its rows and their
columns, every entry's and row's place points at its own column, every row is
some workgroup's, and nothing exceeds what the kernels hold -- over partial
last slices, odd vector chunks, one and two slices per wavefront, the limits of
rows and line widths and one past each, and every way to give a matrix.
"""
import ctypes
import time

import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W

pytestmark = pytest.mark.sym_expanded
EMPTY = 65535


def banded(n, width):
    """Rows of `width` consecutive columns (fewer at the ends) around the diagonal."""
    i = np.arange(n)
    col = i[:, None] + np.arange(width) - width // 2
    ok = (col >= 0) & (col < n)
    ptr = np.zeros(n + 1, np.int32)
    ptr[1:] = np.cumsum(ok.sum(axis=1))
    return ptr, col[ok].astype(np.int32)


def check(fmt, arrs, ptr, idx, base=0):
    """The plan of `arrs` against the full rows ptr / idx."""
    n = len(ptr) - 1
    st, p = cgmi.cg_analyze_resident(fmt, n, *arrs, index_base=base)
    assert st == 0
    if p["wgs"] == 0:
        return p
    G, nsig, ns, off = p["wgs"], p["product_wgs"], p["slices"], p["slice_off"].astype(np.int64)
    wide = p["threads"] == 512
    assert p["threads"] in (256, 512) and 1 <= G <= 256 and ns == (n + 63) // 64
    assert G == ((p["vec_wgs"] + 1) // 2 if wide else p["vec_wgs"]) and nsig <= (1024 if wide else 256)
    assert p["vec_wgs"] * p["vec_chunk"] >= n and p["vec_chunk"] <= 256 * p["slices_per_wave"]
    assert p["slices_per_wave"] <= (2 if wide else 1) and p["width"] <= (16 if wide else 32)
    lens = np.diff(ptr)
    assert p["width"] == lens.max()
    assert p["max_columns"] == np.diff(p["col_ptr"]).max()
    assert p["max_columns"] <= ((10 if p["slices_per_wave"] == 2 else 6) * 384 if wide else 16 * 192)
    runs = np.arange(nsig + 1, dtype=np.int64) * ns // nsig
    assert np.diff(runs).min() >= 1 and np.diff(runs).max() <= 4
    want_entry = np.full(p["positions"], EMPTY, np.int64)
    seen = 0
    for b in range(G):
        s0, s1 = runs[b * nsig // G], runs[(b + 1) * nsig // G]
        assert s1 - s0 <= p["threads"] // 64 * p["slices_per_wave"]
        r0, r1 = s0 * 64, min(n, s1 * 64)
        assert r0 == seen
        seen = r1
        rows = np.arange(r0, r1)
        cols = idx[ptr[r0]:ptr[r1]]
        lst = p["col"][p["col_ptr"][b]:p["col_ptr"][b + 1]]
        assert np.array_equal(lst, np.union1d(rows, cols))
        assert np.array_equal(lst[p["own"][r0:r1]], rows)
        r = np.repeat(rows, lens[r0:r1])
        k = np.arange(ptr[r0], ptr[r1]) - ptr[r]
        want_entry[off[r // 64] + 64 * k + r % 64] = 8 * np.searchsorted(lst, cols)
    assert seen == n
    assert np.array_equal(p["entry"], want_entry)
    return p


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 1000, 30001, 65535, 65536, 65537, 70001, 131072, 131073,
                               200001, 262144])
def test_row_ranges(n, monkeypatch):
    if n <= 2:  # (by default not sliced: nearly all padding)
        monkeypatch.setenv("CGMI_ROW_LAYOUT", "slices")
    a = banded(n, 3)
    p = check("csr", a, *a)
    assert p["wgs"] > 0 and p["threads"] == (256 if n <= 65536 else 512)


def test_past_the_row_limit():
    a = banded(262145, 3)
    assert check("csr", a, *a)["wgs"] == 0


@pytest.mark.parametrize("n,last", [(2000, 32), (70001, 16)])
def test_width_limits(n, last, monkeypatch):
    monkeypatch.setenv("CGMI_ROW_LAYOUT", "slices")
    for width in (last - 1, last, last + 1):
        a = banded(n, width)
        assert (check("csr", a, *a)["wgs"] > 0) == (width <= last), width


@pytest.mark.parametrize("n,reach", [(8000, 3072), (70001, 2304), (200001, 3840)])
def test_column_limits(n, reach):
    """A workgroup whose column list is as long as the kernel holds, and one longer."""
    st, p = cgmi.cg_analyze_resident("csr", n, *banded(n, 3))
    rows = int(p["col_ptr"][2] - p["col_ptr"][1]) - 2  # rows of workgroup 1 (not the first: columns on both sides)
    first = int(p["col"][p["col_ptr"][1]]) + 1
    for extra, ok in ((0, True), (1, False)):
        need = reach - (rows + 2) + extra  # columns beyond the band, spread over its rows
        ptr, idx = banded(n, 3)
        far = np.setdiff1d(np.arange(n), np.arange(first - 1, first + rows + 1))[:need]
        row = first + np.arange(need) % rows
        key = np.unique(np.concatenate([np.repeat(np.arange(n, dtype=np.int64), np.diff(ptr)) * n + idx,
                                        row * np.int64(n) + far]))
        col = (key % n).astype(np.int32)
        ptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int32)
        p = check("csr", (ptr, col), ptr, col)
        assert (p["wgs"] > 0) == ok and (not ok or p["max_columns"] == reach), (extra, p["wgs"])


@pytest.mark.parametrize("shape", [(7, 5, 3), (33, 31, 29), (43, 41, 40), (63, 64, 61)])
def test_every_format(shape):
    s = W.fem_p1_system(*shape, seed=2, with_rhs=False)
    full = (s.rowptr, s.col)
    up = W.upper_triangle(s.rowptr, s.col, s.val)[:2]
    plans = [check("csr", full, *full), check("symcsr", up, *full), check("csc", full, *full),
             check("csr", (s.rowptr + 1, s.col + 1), *full, base=1)]
    for p in plans:
        assert p["wgs"] > 0
        assert all(np.array_equal(p[k], plans[0][k]) for k in p)


def test_columns_of_a_nonsymmetric_matrix():
    ptr, idx, val = W.banded_sparse(9000, 40, density=0.2, seed=4, empty=50)
    n = len(ptr) - 1
    rows = W.transpose_csr(n, n, ptr, idx, val)
    check("csc", (ptr, idx), *rows[:2])


def test_errors():
    a = banded(10, 3)
    assert cgmi.cg_analyze_resident("csr", -1, *a)[0] == cgmi.CG_ERR_ARG
    assert cgmi.cg_analyze_resident("csr", 10, a[0], a[1][::-1].copy())[0] == cgmi.CG_ERR_STRUCTURE
    assert cgmi.cg_analyze_resident("csr", 0, np.zeros(1, np.int32), np.zeros(0, np.int32))[1]["wgs"] == 0


def test_no_host_memory(monkeypatch):
    s = W.fem_p1_system(43, 41, 40, seed=2, with_rhs=False)
    up = W.upper_triangle(s.rowptr, s.col, s.val)[:2]
    monkeypatch.setenv("CGMI_CHOICE_FAILS", "host")
    for fmt, a in (("csr", (s.rowptr, s.col)), ("csc", (s.rowptr, s.col)), ("symcsr", up)):
        st, p = cgmi.cg_analyze_resident(fmt, s.n, *a)
        assert st == 0 and p["wgs"] == 0, fmt


def test_one_plan_where_one_is_used():
    """A symmetric system that runs by rows alone is planned by rows alone: the
    compact blocks, which take many times as long to grow, are left out."""
    s = W.fem_p1_system(61, 59, 57, seed=1, with_rhs=False)
    ptr, idx = W.upper_triangle(s.rowptr, s.col, s.val)[:2]
    plan = cgmi.cg_resident_plan()
    p, i = (a.ctypes.data_as(ctypes.c_void_p) for a in (ptr, idx))

    def rows():
        st = cgmi.load().cg_analyze_resident(cgmi.CG_FMT_SYM_CSR, s.n, p, i, 0, ctypes.byref(plan), *[None] * 5)
        assert st == 0 and plan.wgs > 0

    def best(f):
        out = []
        for _ in range(5):
            t = time.perf_counter()
            f()
            out.append(time.perf_counter() - t)
        return min(out)
    assert best(rows) < 0.5 * best(lambda: cgmi.cg_analyze("symcsr", s.n, ptr, idx))  # (0.1; both plans: 1.0)
