"""The layout by rows beside CSC panels and compact symmetric blocks is a
choice, and so is the resident solve of sliced rows: where the host or the
device has no memory for it, a handle is made without it, and products, solves
and new values have the bits of a handle that never had one.
"""
import ctypes

import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.sym_expanded]


@pytest.mark.parametrize("where", ["host", "device"])
@pytest.mark.parametrize("kind", ["csr", "csc_small", "csc", "csc_mixed", "symcsr", "symcsr_small", "lower"])
def test_create_without_memory_for_choices(kind, where, monkeypatch):
    s = W.fem_p1_system(*((13, 12, 11) if "small" in kind else (43, 42, 40)), nu_iron=0.5, seed=1)
    fmt, arrs, flags = kind[:3], (s.rowptr, s.col, s.val), 0
    without = "CGMI_RESIDENT" if kind in ("csr", "symcsr_small") else "CGMI_SYM_EXPAND"
    if kind in ("symcsr", "symcsr_small", "lower"):
        fmt, arrs = "symcsr", W.upper_triangle(*arrs)
        if kind == "lower":
            arrs, flags = W.transpose_csr(s.n, s.n, *arrs), cgmi.CG_LOWER
    x = to_dev(W.uniform_vector(s.n, seed=2))
    out, size = [], []
    for env in ((without, "0"), ("CGMI_CHOICE_FAILS", where), (None, None)):
        if env[0]:
            monkeypatch.setenv(*env)
        with cgmi.Solver(fmt, *arrs, flags=flags, mixed=kind == "csc_mixed") as S:
            res = [S.spmv(x), S.spmv_static(x), S.solve(to_dev(s.b), tol=1e-9)[0]]
            S.set_values(to_dev(arrs[2] * 1.5))
            res += [S.spmv(x), S.solve(to_dev(s.b), tol=1e-9)[0], S.pattern_grad(x, x)]
            out.append([r.cpu().numpy() for r in res])
            size.append(S.stats()["device_bytes"])
            say(f"{kind} {env}: {size[-1]} bytes, path {S.report()}")
        if env[0]:
            monkeypatch.delenv(env[0])
    assert size[0] == size[1] and size[2] != size[0]
    for a, b in zip(*out[:2]):
        assert np.array_equal(a, b)


def host_bytes_held(S):
    """What closing the handle gives back to the system."""
    libc = ctypes.CDLL("libc.so.6")

    def resident_bytes():
        libc.malloc_trim(0)
        return int(open("/proc/self/statm").read().split()[1]) * 4096
    before = resident_bytes()
    S.close()
    return before - resident_bytes()


def test_host_memory_of_the_rows_plan(monkeypatch):
    """A handle with the layout by rows keeps no more on the host than one
    without: the plan (6 bytes a position, 5.8 million here; 23 MB held) is given
    back once it is on the device."""
    s = W.fem_p1_system(74, 73, 72, seed=1, with_rhs=False)
    monkeypatch.setenv("CGMI_SYM_EXPAND", "0")
    alone = host_bytes_held(cgmi.Solver("csc", s.rowptr, s.col, s.val))
    monkeypatch.delenv("CGMI_SYM_EXPAND")
    both = host_bytes_held(cgmi.Solver("csc", s.rowptr, s.col, s.val))
    say(f"host bytes held by a handle: {alone} without rows, {both} with")
    assert both <= alone + (12 << 20)
