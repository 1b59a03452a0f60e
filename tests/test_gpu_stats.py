"""A handle's summary describes the layouts it holds: the rows that its product
runs on where there are any, the storage format's blocks only while something
runs on them, and bytes that the allocations account for.
"""
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
