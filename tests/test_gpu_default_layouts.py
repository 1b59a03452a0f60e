"""The tests of products, solves, new values and mixed precision of CSC and
symmetric matrices, once more on the layouts that the library chooses by
itself: elsewhere CGMI_SYM_EXPAND=0 keeps the panels and the scatter plans on
small systems too (conftest.py), here full rows are laid out where they are by
default.
"""
import inspect

import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests import test_gpu_adjoint as adj
from tests import test_gpu_cg as cg
from tests import test_gpu_mixed as mixed
from tests import test_gpu_spmv as spmv
from tests import test_gpu_values as values
from tests.gpu_util import say, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.sym_expanded]
SYM, CSC = cgmi.CG_FMT_SYM_CSR, cgmi.CG_FMT_CSC
CASES = [(f, dict(fmt=fmt)) for fmt in (SYM, CSC)
         for f in (spmv.test_fem_small, spmv.test_fem_paper_sized, spmv.test_one_based, spmv.test_tiny_and_empty,
                   spmv.test_deterministic_and_stream_ordered, cg.test_random_spd, cg.test_fem_paper_sized,
                   cg.test_early_iterates_match, cg.test_nonzero_start, cg.test_deterministic, cg.test_status_paths,
                   cg.test_breakdown_on_indefinite, mixed.test_mixed_paper_sized)]
CASES += [(values.test_values_and_gradients_exact, dict(fmt=fmt, layout=layout))
          for fmt in ("symcsr", "lower", "csc") for layout in ("", "slices")]
CASES += [(f, {}) for f in (spmv.test_csc_is_a_true_scatter, spmv.test_sym_random_spd,
                            spmv.test_lower_triangle_input_matches_full_product, adj.test_pattern_grad_bit_exact,
                            adj.test_set_values_matches_fresh_handle, adj.test_set_values_mixed)]
CASES += [(spmv.test_ragged_nonsymmetric, dict(fmt=CSC, layout=layout)) for layout in ("rows", "slices")]
CASES += [(spmv.test_csc_panels, dict(case=case, layout=layout)) for layout in ("rows", "slices")
          for case in ("fem_two_colours", "banded_empty_lines", "dense_row")]


@pytest.mark.parametrize("test,args", CASES, ids=["-".join([f.__name__[5:], *map(str, a.values())]) for f, a in CASES])
def test_again(test, args, monkeypatch):
    if "monkeypatch" in inspect.signature(test).parameters:
        args = dict(args, monkeypatch=monkeypatch)
    test(**args)


@pytest.mark.parametrize("fmt", ["csc", "symcsr"])
def test_layouts_are_the_defaults(fmt):
    """What the handles of these cases hold: rows alone where solves can be
    resident; else the format's own."""
    s = W.fem_p1_system(12, 11, 10, seed=1)
    full = (s.rowptr, s.col, s.val)
    arrs = W.upper_triangle(*full) if fmt == "symcsr" else full
    with cgmi.Solver(fmt, *arrs) as S:
        S.solve(to_dev(s.b), tol=1e-8)
        st, r = S.stats(), S.report()
        say(f"default {fmt}: {st} {r}")
        assert st["slots"] == 0 and st["slices"] == 2 and r["path"] == cgmi.CG_PATH_RESIDENT
    n = 300
    rows = W.random_sparse(n, density=0.02, seed=7, empty_rows=20, long_rows=2, long_len=280)
    ptr, idx, val = W.transpose_csr(n, n, *rows)
    with cgmi.Solver("csc", ptr, idx, val) as S:  # too ragged for slices
        assert S.stats()["slots"] > 0
        assert np.isfinite(S.spmv(to_dev(W.uniform_vector(n, seed=8))).cpu().numpy()).all()
