"""Which way a solve ran (cg_get_solve_report): the resident kernel wherever one
is planned, launches past each limit, repeated by launches after a wait that
ran out -- so that the comparisons of the paths' bits compare two paths.
"""
import threading

import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say, to_dev
from tests.test_gpu_resident import tridiagonal

pytestmark = [pytest.mark.gpu, pytest.mark.sym_expanded]
RESIDENT, LAUNCHES, REPEATED = cgmi.CG_PATH_RESIDENT, cgmi.CG_PATH_LAUNCHES, cgmi.CG_PATH_REPEATED


@pytest.mark.parametrize("n", [1, 64, 257, 30001, 65536, 65537, 131073, 262144, 262145])
def test_rows(n, monkeypatch):
    if n == 1:  # (by default not sliced: nearly all padding)
        monkeypatch.setenv("CGMI_ROW_LAYOUT", "slices")
    say(f"path of tridiagonal n={n}")
    arrs = tridiagonal(n)
    with cgmi.Solver("csr", *arrs) as S:
        assert S.report()["path"] == cgmi.CG_PATH_NONE
        S.solve(to_dev(W.uniform_vector(n, seed=1)), tol=1e-10, maxit=50)
        r = S.report()
    planned = cgmi.cg_analyze_resident("csr", n, *arrs[:2])[1]["wgs"]
    assert r["resident_wgs"] == planned and (planned > 0) == (n <= 262144)
    assert r["path"] == (RESIDENT if planned else LAUNCHES) and (r["graphs"] > 0) == (not planned)


@pytest.mark.parametrize("per_row,path", [(16, RESIDENT), (40, LAUNCHES)])
def test_widths(per_row, path, monkeypatch):
    monkeypatch.setenv("CGMI_ROW_LAYOUT", "slices")
    arrs = W.random_spd_sparse(2000, density=(per_row - 1) / 2000, seed=per_row)
    with cgmi.Solver("csr", *arrs) as S:
        S.solve(to_dev(W.uniform_vector(2000, seed=3)), tol=1e-10, maxit=300)
        assert S.report()["path"] == path


@pytest.mark.parametrize("fmt", ["csr", "symcsr", "csc"])
@pytest.mark.parametrize("shape", [(21, 19, 17), (47, 45, 43)])
def test_formats(fmt, shape, monkeypatch):
    s = W.fem_p1_system(*shape, nu_iron=0.5, seed=4)
    arrs = W.upper_triangle(s.rowptr, s.col, s.val) if fmt == "symcsr" else (s.rowptr, s.col, s.val)
    for fused, path in ((None, RESIDENT), ("0", LAUNCHES)):
        if fused:
            monkeypatch.setenv("CGMI_FUSED", fused)
        with cgmi.Solver(fmt, *arrs, mixed=fmt == "csr") as S:
            S.solve(to_dev(s.b), tol=1e-8)
            assert S.report()["path"] == path
            if fmt == "csr":
                S.solve_mixed(to_dev(s.b), tol=1e-8)
                assert S.report()["path"] == LAUNCHES and S.report()["graphs"] > 0


def test_wait_that_ran_out(monkeypatch):
    s = W.fem_p1_system(16, 15, 14, seed=8)
    monkeypatch.setenv("CGMI_RESIDENT_WAIT", "-1")
    with cgmi.Solver("csr", s.rowptr, s.col, s.val) as S:
        S.solve(to_dev(s.b), tol=1e-10)
        assert S.report()["path"] == REPEATED and S.report()["graphs"] > 0


def test_two_solves_share_the_device():
    """180 workgroups each: never two resident at a time, so none ever gives up."""
    import torch
    s = W.fem_p1_system(36, 36, 35, seed=10)
    b = to_dev(s.b)
    torch.cuda.synchronize()
    paths = {0: [], 1: []}

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()), cgmi.Solver("csr", s.rowptr, s.col, s.val) as S:
            for _ in range(20):
                S.solve(b)
                paths[k].append(S.report()["path"])
            torch.cuda.current_stream().synchronize()
    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    say(f"paths {paths}")
    assert set(paths[0] + paths[1]) <= {RESIDENT, LAUNCHES}
    assert RESIDENT in paths[0] + paths[1]
    assert np.all([len(p) == 20 for p in paths.values()])


def test_resident_again_after_a_wait_that_ran_out(monkeypatch):
    """One missed wait costs some solves by launches, not the handle's life; and
    while waits go on running out, most solves do not try."""
    import time  # (a repeated solve loses some 0.1 ms, so the solves are kept shorter than the pause after it)
    s = W.fem_p1_system(16, 15, 14, seed=8)
    b = to_dev(s.b)
    with cgmi.Solver("csr", s.rowptr, s.col, s.val) as S:
        ref = S.solve(b, tol=1e-10, maxit=20)
        assert S.report()["path"] == RESIDENT
        monkeypatch.setenv("CGMI_RESIDENT_WAIT", "-1")
        paths = []
        for _ in range(50):
            x, info = S.solve(b, tol=1e-10, maxit=20)
            paths.append(S.report()["path"])
        say(f"paths while waits run out: {paths}")
        assert paths[0] == REPEATED and set(paths) == {REPEATED, LAUNCHES}
        assert paths.count(REPEATED) <= len(paths) // 2
        monkeypatch.delenv("CGMI_RESIDENT_WAIT")
        end = time.monotonic() + 30
        while S.report()["path"] != RESIDENT and time.monotonic() < end:
            x, info = S.solve(b, tol=1e-10, maxit=20)
        assert S.report()["path"] == RESIDENT
        assert np.array_equal(x.cpu().numpy(), ref[0].cpu().numpy()) and info["iters"] == ref[1]["iters"]
