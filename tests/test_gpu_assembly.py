"""Assembly of A(nu) where its contribution lists are unusual: a fan of
elements around one edge (lists longer than the 2048 contributions one
workgroup holds, 1 and 2 below and above it), a single element, and points
tied to one unknown (several vertices of an element on one row).  Checked
entry by entry against a plain sum in numpy over the device's own element
matrices (which tests/test_gpu_adjoint.py checks); each value is a sum of m
products, so its rounding error is within (m + 40) 2^-53 of the sum of their
absolute values.
"""
import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def fan(m):
    """m tetrahedra around the edge (0, 1), their ring closed."""
    a = 2 * np.pi * np.arange(m) / m
    ring = np.stack([np.cos(a), np.sin(a), np.zeros(m)], axis=1)
    pts = np.concatenate([[[0.0, 0.0, -1.0], [0.0, 0.0, 1.0]], ring])
    i = np.arange(m)
    tets = np.stack([0 * i, 0 * i + 1, 2 + i, 2 + (i + 1) % m], axis=1)
    return pts, tets.astype(np.int32)


def cases():
    for m in (3, 2046, 2047, 2048, 2049, 2051):
        pts, tets = fan(m)
        yield f"fan{m}", pts, tets, np.arange(len(pts), dtype=np.int32), len(pts)
    pts, tets = fan(7)
    one = np.array([[0, 1, 2, 3]], np.int32)
    yield "one", pts[:4], one, np.arange(4, dtype=np.int32), 4
    yield "one_fixed", pts[:4], one, np.array([0, -1, 1, -1], np.int32), 2
    tied = np.arange(len(pts), dtype=np.int32) // 2    # vertices in pairs on one unknown
    yield "tied", pts, tets, tied, int(tied.max()) + 1


def test_assembly_lists():
    for name, pts, tets, dof, n in cases():
        say(name)
        nu = np.random.default_rng(1).uniform(0.5, 2.0, size=len(tets))
        with cgmi.FemOperator(pts, tets, dof, n) as F:
            rp, col = F.pattern()
            got = F.assemble(to_dev(nu)).cpu().numpy()
        # the element matrices, one by one: the same elements with no shared
        # vertex and nu = 1 (slivers are ill conditioned, so another evaluation
        # of K would differ by more than the sums under test)
        m4 = 4 * len(tets)
        with cgmi.FemOperator(pts[tets].reshape(m4, 3), np.arange(m4).reshape(-1, 4), np.arange(m4), m4) as F:
            K = F.assemble(to_dev(np.ones(len(tets)))).cpu().numpy().reshape(-1, 4, 4)
        mag = np.sqrt(np.einsum("eaa->ea", K))
        S, B, M = np.zeros((n, n)), np.zeros((n, n)), np.zeros((n, n), np.int64)
        for a in range(4):
            for b in range(4):
                i, j = dof[tets[:, a]], dof[tets[:, b]]
                ok = (i >= 0) & (j >= 0)
                np.add.at(S, (i[ok], j[ok]), (nu * K[:, a, b])[ok])
                np.add.at(B, (i[ok], j[ok]), (nu * mag[:, a] * mag[:, b])[ok])
                np.add.at(M, (i[ok], j[ok]), 1)
        line = np.repeat(np.arange(n), np.diff(rp))
        assert np.array_equal(M > 0, np.isin(np.arange(n * n), line * n + col).reshape(n, n)), name
        # two evaluations, each within the bound of the exact sum
        assert np.all(np.abs(got - S[line, col]) <= 2 * (M[line, col] + 40) * 2.0 ** -53 * B[line, col]), name
        A = np.zeros((n, n))
        A[line, col] = got
        assert np.array_equal(A, A.T), name
