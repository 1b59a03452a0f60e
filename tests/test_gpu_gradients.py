"""Value gradients at each form of the kernel, chosen by the mean and the
longest line: lines of one or two entries (a thread each), then passes of 3, 4,
6, 8 and 16 entries a lane; empty lines, line counts around 64, one long line
among short ones.  Exact: the bits of the rounded products.
"""
import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def lines(n, lens, seed, upper):
    """Lines of the given numbers of random ascending columns (upper: from the diagonal on, which each holds)."""
    g = np.random.default_rng(seed)
    col = []
    for i, k in enumerate(lens):
        if upper:
            rest = g.choice(np.arange(i + 1, n), size=min(k - 1, n - 1 - i), replace=False)
            col.append(np.sort(np.concatenate([[i], rest])))
        else:
            col.append(np.sort(g.choice(n, size=min(k, n), replace=False)))
    ptr = np.concatenate([[0], np.cumsum([len(c) for c in col])])
    return ptr.astype(np.int32), np.concatenate(col).astype(np.int32)


@pytest.mark.parametrize("fmt", ["csr", "csc", "symcsr"])
@pytest.mark.parametrize("mean", [1, 2, 3, 4, 5, 6, 7, 8, 9, 17, "long2", "long3"])
def test_exact(fmt, mean):
    for n in (63, 64, 65, 321):
        g = np.random.default_rng(n)
        if isinstance(mean, str):  # one line of a run of its own
            lens = np.full(n, int(mean[4:]) - 1)
            lens[n // 3] = n
        else:  # lengths around the mean, empty lines among them where the format has them
            lens = np.maximum(g.integers(0, 2 * mean + 1, size=n), 1 if fmt == "symcsr" else 0)
            if mean == 1:
                lens[:] = 1
        ptr, col = lines(n, lens, n, fmt == "symcsr")
        say(f"gradient {fmt} {mean} n={n} nnz={len(col)} longest={np.diff(ptr).max()}")
        lam, x = g.uniform(-1, 1, size=n), g.uniform(-1, 1, size=n)
        try:
            S = cgmi.Solver(fmt, ptr, col, np.ones(len(col)))
        except cgmi.CgError as e:
            assert e.status == cgmi.CG_ERR_UNSUPPORTED and fmt == "symcsr"
            continue
        with S:
            got = S.pattern_grad(to_dev(lam), to_dev(x)).cpu().numpy()
        line = np.repeat(np.arange(n), np.diff(ptr))
        i, j = (col, line) if fmt == "csc" else (line, col)
        ref = -(lam[i] * x[j])
        if fmt == "symcsr":
            ref = np.where(i == j, ref, -(lam[i] * x[j] + lam[j] * x[i]))
        assert np.array_equal(got, ref)


def test_short_lines_take_no_longer_than_their_bytes():
    """A million lines of two entries, against a product of two vectors of as
    many values (which moves as much): 1.5 times as long; 3.4 in passes of eight
    entries a lane."""
    import time

    import torch
    n = 1000000
    i = np.arange(n, dtype=np.int32)
    ptr = np.minimum(2 * np.arange(n + 1), 2 * n - 1).astype(np.int32)
    col = np.stack([i, i + 1], axis=1).reshape(-1)[:-1]
    x, out = to_dev(W.uniform_vector(n, seed=1)), to_dev(np.zeros(len(col)))
    a = to_dev(W.uniform_vector(len(col), seed=2))

    def us(f):
        best = []
        for _ in range(20):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(50):
                f()
            torch.cuda.synchronize()
            best.append((time.perf_counter() - t) / 50 * 1e6)
        return min(best)
    with cgmi.Solver("symcsr", ptr, col, np.where(np.diff(col, prepend=-1) >= 0, 2.5, -1.0)) as S:
        got, ref = us(lambda: S.pattern_grad(x, x, out)), us(lambda: torch.mul(a, a, out=out))
    say(f"gradient {got:.1f} us, product of vectors {ref:.1f} us")
    assert got <= 2.3 * ref
