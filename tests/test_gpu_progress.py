"""Solves that the host follows through reports of the iterations (graphs of
launches; several systems in a batch), stopped at every place relative to a
graph's end and to the reports: a solve cut at maxit = k does k iterations and
leaves the iterate that a solve cut one iteration at a time leaves -- exactly,
since graphs of any length run the same kernels.  And the product over slices
with 16 positions in flight, which has the bits of the one with 8.
"""
import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say, to_dev
from tests.test_gpu_batch import small_batch

pytestmark = pytest.mark.gpu
CUTS = (0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33)


@pytest.mark.parametrize("kind", ["csr", "symcsr", "fused", "mixed"])
def test_solve_cut_anywhere(kind, monkeypatch):
    monkeypatch.setenv("CGMI_RESIDENT", "0")
    monkeypatch.setenv("CGMI_FUSED", "1" if kind == "fused" else "0")
    s = W.fem_p1_system(13, 11, 9, seed=3)
    arrs = W.upper_triangle(s.rowptr, s.col, s.val) if kind == "symcsr" else (s.rowptr, s.col, s.val)
    fmt, b = ("symcsr" if kind == "symcsr" else "csr"), to_dev(s.b)
    out = {}
    for batch in (1, 2, 5, 32):
        with cgmi.Solver(fmt, *arrs, batch=batch, mixed=kind == "mixed") as S:
            for cut in CUTS:
                if kind == "mixed":
                    x, info = S.solve_mixed(b, tol=1e-30, maxit=cut, inner_tol=1e-3)
                else:
                    x, info = S.solve(b, tol=1e-30, maxit=cut)
                say(f"{kind} batch {batch} cut {cut}: {info}")
                assert info["status"] == cgmi.CG_NOT_CONVERGED and info["iters"] == cut
                ref = out.setdefault(cut, x.cpu().numpy())
                assert np.array_equal(ref, x.cpu().numpy()), (batch, cut)
            x, info = S.solve(b, tol=1e-10, maxit=5000)  # and one to its end, on the same reports
            assert info["status"] == cgmi.CG_OK
            z, info = S.solve(b * 0, tol=1e-10, maxit=5000)
            assert info["status"] == cgmi.CG_OK and info["iters"] == 0 and not z.any()


@pytest.mark.parametrize("lanes", ["0", "8", "1"])
@pytest.mark.parametrize("nrhs", [1, 2, 4])
def test_batch_cut_anywhere(nrhs, lanes, monkeypatch):
    monkeypatch.setenv("CGMI_BATCH_LANES", lanes)
    systems, B = small_batch(nrhs)
    so, ptr, col, val = W.block_diagonal(systems)
    B[so[2]:so[3]] = 0.0  # a system that never starts
    with cgmi.Batch(so, ptr, col, val, nrhs=nrhs) as bt:
        X, _, iters, stat = bt.solve(to_dev(B), tol=1e-10, maxit=20000)
        assert (stat == 0).all() and (iters[2] == 0).all()
        for cut in CUTS:
            Y, _, it, st = bt.solve(to_dev(B), tol=1e-10, maxit=cut)
            assert np.array_equal(it, np.minimum(iters, cut)), cut
            assert np.array_equal(st, np.where(iters <= cut, 0, cgmi.CG_NOT_CONVERGED)), cut
        # pairs that stop early keep their solution while others go on
        cut = int(np.median(iters))
        Y, _, it, st = bt.solve(to_dev(B), tol=1e-10, maxit=cut)
        X, Y = X.cpu().numpy().reshape(-1, nrhs), Y.cpu().numpy().reshape(-1, nrhs)
        for s in range(len(systems)):
            for r in range(nrhs):
                if iters[s, r] <= cut:
                    assert np.array_equal(X[so[s]:so[s + 1], r], Y[so[s]:so[s + 1], r]), (s, r)


@pytest.mark.parametrize("nrhs", [1, 2])
@pytest.mark.parametrize("col16", ["0", "1"])
def test_batch_deep_slices_same_bits(nrhs, col16, monkeypatch):
    monkeypatch.setenv("CGMI_BATCH_LANES", "1")
    monkeypatch.setenv("CGMI_COL16", col16)
    systems, B = small_batch(nrhs)  # (FEM rows of up to 15 entries; random ones of odd, even and more than 16)
    for k, dens in enumerate((0.02, 0.2)):
        systems.append(W.random_spd_sparse(131, density=dens, seed=40 + k))
        B = np.concatenate([B, np.random.default_rng(k).uniform(-1, 1, size=(131, nrhs))])
    so, ptr, col, val = W.block_diagonal(systems)
    out = {}
    for deep in ("0", "1"):
        monkeypatch.setenv("CGMI_BATCH_DEEP", deep)
        with cgmi.Batch(so, ptr, col, val, nrhs=nrhs) as bt:
            Y = bt.spmm(to_dev(B)).cpu().numpy()
            X, info, iters, stat = bt.solve(to_dev(B), tol=1e-10, maxit=20000)
            out[deep] = (Y, X.cpu().numpy(), iters)
    assert all(np.array_equal(a, b) for a, b in zip(out["0"], out["1"]))
