"""Solves by launches keep the GPU fed: the next graph of iterations is on its
way while iterations of the one before are still to come -- with three kernels
an iteration and with two (small systems that cannot be resident), and in the
inner solves of mixed precision.
"""
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.sym_expanded]


@pytest.mark.parametrize("batch", [8, 32])
@pytest.mark.parametrize("kind", ["two kernels", "three kernels", "mixed"])
def test_graphs_overlap(kind, batch, monkeypatch):
    monkeypatch.setenv("CGMI_RESIDENT", "0")
    if kind != "two kernels":
        monkeypatch.setenv("CGMI_FUSED", "0")
    s = W.fem_p1_system(31, 30, 29, nu_iron=1e-4, seed=3)
    with cgmi.Solver("csr", s.rowptr, s.col, s.val, batch=batch, mixed=kind == "mixed") as S:
        if kind == "mixed":
            S.solve_mixed(to_dev(s.b), tol=1e-30, maxit=640, inner_tol=1e-12, max_outer=1)
        else:
            S.solve(to_dev(s.b), tol=0.0, maxit=640)
        r = S.report()
    say(f"{kind} batch {batch}: {r}")
    assert r["path"] == cgmi.CG_PATH_LAUNCHES and r["graphs"] >= 20
    assert 2 * r["ahead"] >= r["graphs"]  # (each but the first, unless the host is held up)
