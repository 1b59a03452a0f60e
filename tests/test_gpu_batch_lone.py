"""Lone products of batches whose systems have more row blocks or slices than a
solve gives workgroups to (1024): their own split, every schedule, against the
oracle; the slices' bits do not depend on the split; and a solve after a product.
"""
import numpy as np
import pytest

import oracle
from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import SPMV_TOL, say, spmv_bound, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [1, 2, 4])
def test_products_of_large_systems(nrhs, monkeypatch):
    big, small = W.fem_p1_system(47, 45, 43, nu_iron=0.5, seed=1), W.fem_p1_system(5, 4, 3, nu_iron=0.5, seed=2)
    so, ptr, col, val = W.block_diagonal([(s.rowptr, s.col, s.val) for s in (small, big, small)])
    n = int(so[-1])
    X = np.random.default_rng(3).uniform(-1, 1, size=(n, nrhs))
    want = [oracle.spmv(cgmi.CG_FMT_CSR, ptr, col, val, np.ascontiguousarray(X[:, r])) for r in range(nrhs)]
    bound = [SPMV_TOL * spmv_bound(cgmi.CG_FMT_CSR, ptr, col, val, X[:, r]) for r in range(nrhs)]
    bits = {}
    for lanes, deep in (("0", "0"), ("8", "0"), ("16", "0"), ("1", "0"), ("1", "1")):
        monkeypatch.setenv("CGMI_BATCH_LANES", lanes)
        monkeypatch.setenv("CGMI_BATCH_DEEP", deep)
        with cgmi.Batch(so, ptr, col, val, nrhs=nrhs) as b:
            say(f"lone products nrhs={nrhs} lanes={lanes} deep={deep}")
            Y = b.spmm(to_dev(X)).cpu().numpy().reshape(n, nrhs)
            S, info, iters, stat = b.solve(to_dev(Y), tol=1e-8, maxit=3000)
            assert np.array_equal(Y, b.spmm(to_dev(X)).cpu().numpy().reshape(n, nrhs))
        for r in range(nrhs):
            assert np.all(np.abs(Y[:, r] - want[r]) <= bound[r])
        assert (stat == 0).all()
        if lanes == "1":
            bits[deep] = Y
    assert np.array_equal(bits["0"], bits["1"])
