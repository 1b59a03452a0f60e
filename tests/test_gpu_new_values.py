"""New values of systems whose graph is many pockets (compact blocks of one line
and up): the layout's bits, and about as fast as the values can be copied.
"""
import time

import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def chains(n, length):
    """Upper triangle of separate chains of `length` lines."""
    i = np.arange(n)
    last = (i % length == length - 1) | (i == n - 1)
    ptr = np.concatenate([[0], np.cumsum(np.where(last, 1, 2))]).astype(np.int32)
    col = np.empty(ptr[-1], np.int32)
    col[ptr[:-1]] = i
    col[ptr[:-1][~last] + 1] = i[~last] + 1
    return ptr, col


def best_us(f):
    import torch
    out = []
    for _ in range(10):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(30):
            f()
        torch.cuda.synchronize()
        out.append((time.perf_counter() - t) / 30 * 1e6)
    return min(out)


@pytest.mark.parametrize("length", [1, 2, 63, 255, 256, 257, 1000])
@pytest.mark.parametrize("lower", [False, True])
def test_bits(length, lower):
    n = 66000
    ptr, col = chains(n, length)
    g = np.random.default_rng(length)
    old, new = g.uniform(1, 2, size=(2, len(col)))
    flags = 0
    if lower:
        ptr, col, old = W.transpose_csr(n, n, ptr, col, old)
        flags = cgmi.CG_LOWER
    x = to_dev(W.uniform_vector(n, seed=1))
    say(f"chains of {length}, lower {lower}")
    with cgmi.Solver("symcsr", ptr, col, old, flags=flags) as S, cgmi.Solver("symcsr", ptr, col, new, flags=flags) as F:
        S.set_values(to_dev(new))
        assert np.array_equal(S.spmv(x).cpu().numpy(), F.spmv(x).cpu().numpy())


@pytest.mark.parametrize("length", [1, 4, 16])
def test_time_of_many_small_blocks(length):
    import torch
    n = 1 << 20
    ptr, col = chains(n, length)
    v = to_dev(np.random.default_rng(1).uniform(1, 2, size=len(col)))
    out = torch.empty_like(v)
    with cgmi.Solver("symcsr", ptr, col, v.cpu().numpy()) as S:
        got, copy = best_us(lambda: S.set_values(v)), best_us(lambda: out.copy_(v))
    say(f"chains of {length}: set_values {got:.1f} us, copy {copy:.1f} us")  # (6.5; a workgroup a block 40 to 560)
    assert got <= 3.5 * copy
