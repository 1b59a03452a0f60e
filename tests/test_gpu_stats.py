"""A handle's summary describes the layouts it holds: the rows that its product
runs on where there are any, the storage format's blocks only while something
runs on them, and bytes that the allocations account for.
"""
import numpy as np
import pytest

from paper_1010_4639_amd import cgmi
from paper_1010_4639_amd import workload as W
from tests.gpu_util import say

pytestmark = [pytest.mark.gpu, pytest.mark.sym_expanded]
BLOCKS = ("scatter_blocks", "max_block_entries", "colors", "compact", "slots", "parked")


# fmt, grid, mixed: on rows alone; on rows beside the format's blocks; on the blocks
CASES = [("csc", (13, 12, 11), False, "rows"), ("csc", (43, 42, 40), False, "rows"),
         ("symcsr", (43, 42, 40), False, "rows"), ("csc", (66, 65, 64), False, "beside"),
         ("csc", (43, 42, 40), True, "beside"), ("symcsr", (43, 42, 40), True, "beside"),
         ("symcsr", (66, 65, 64), False, "blocks"), ("symcsr", (13, 12, 11), False, "blocks"),
         ("csr", (43, 42, 40), False, "blocks")]


@pytest.mark.parametrize("fmt,grid,mixed,kind", CASES)
def test_summary(fmt, grid, mixed, kind):
    s = W.fem_p1_system(*grid, seed=1, with_rhs=False)
    full = (s.rowptr, s.col, s.val)
    arrs = W.upper_triangle(*full) if fmt == "symcsr" else full
    own = cgmi.cg_analyze(fmt, s.n, *arrs)[1]
    csr = cgmi.cg_analyze("csr", s.n, *full)[1]  # the rows' plan
    with cgmi.Solver(fmt, *arrs, mixed=mixed) as S:
        st = S.stats()
    say(f"{fmt} {grid} {kind}: {st}")
    assert st["nnz"] == len(arrs[1]) and st["format"] == own["format"] and st["vec_blocks"] == own["vec_blocks"]
    for f in ("spmv_blocks", "slices", "cached_loads", "plan_bytes"):
        assert st[f] == (own if kind == "blocks" else csr)[f], f
    for f in BLOCKS:
        assert st[f] == (0 if kind == "rows" else own[f]), f
    assert st["device_bytes"] >= st["plan_bytes"] + 4 * (s.n + 1) + 4 * len(arrs[1])


@pytest.mark.parametrize("n,kind", [(300000, "blocks"), (200000, "blocks"), (300000, "beside"), (200000, "rows")])
def test_rows_beside_one_panel(n, kind, monkeypatch):
    """Columns in no order are one panel, whose slots are whole rows: no second
    layout, unless solves can be resident (here: rows coupled to the next one and,
    on one panel, the first to the last)."""
    i = np.arange(n)
    if kind == "blocks":
        g = np.random.default_rng(7)
        far = [g.permutation(n) for _ in range(4)]
        pairs = [(f[:-1], f[1:]) for f in far]
    else:
        pairs = [(i[:-1], i[1:])] + ([(i[:1], i[-1:])] if kind == "rows" else [])
    r = np.concatenate([i] + [p[0] for p in pairs] + [p[1] for p in pairs])
    c = np.concatenate([i] + [p[1] for p in pairs] + [p[0] for p in pairs])
    key = np.unique(r.astype(np.int64) * n + c)
    ptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int32)
    col = (key % n).astype(np.int32)
    val = np.where(col == key // n, 9.0, -1.0)
    own = cgmi.cg_analyze("csc", n, ptr, col)[1]
    size = {}
    for expand in ("0", None):
        monkeypatch.setenv("CGMI_SYM_EXPAND", expand) if expand else monkeypatch.delenv("CGMI_SYM_EXPAND")
        with cgmi.Solver("csc", ptr, col, val) as S:
            st = S.stats()
            size[expand] = st["device_bytes"]
    say(f"{n} {kind}: {st}, {size}")
    assert (own["colors"] == 2) == (kind == "beside")
    assert st["slots"] == (0 if kind == "rows" else own["slots"])
    assert (size[None] == size["0"]) == (kind == "blocks")
