"""Sweeps of a coarsest level too large for the precomputed forms, with fewer lanes
a row than its average length asks for (more rows than a full chip's threads hold at
that width), against the oracle.  An odd number of sweeps keeps them one by one; the
bounds are those of one cycle."""
import numpy as np
import pytest

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP32, ENTRY_FP64, B, _close_entries, say  # noqa: F401

pytestmark = pytest.mark.gpu

# 8 lanes by the rows (5 and 7 entries): all resident up to 65,536 rows; and rows of 76
CASES = {"65536 rows": lambda: P.poisson2d(256, 256)[:3], "65792 rows": lambda: P.poisson2d(256, 257)[:3],
         "70x71x67": lambda: P.poisson3d(70, 71, 67)[:3], "elasticity": lambda: P.elasticity3d(15, 2)[:3]}


@pytest.mark.parametrize("max_levels", [1, 2])
@pytest.mark.parametrize("name", list(CASES))
def test_sweeps_of_a_large_coarsest_level(B, ora, name, max_levels):  # noqa: F811
    rp, ci, va = CASES[name]()
    n = len(rp) - 1
    say(f"coarsest sweeps: {name} n={n} nnz={len(ci)} levels={max_levels}")
    r = P.uniform_rhs(n, 4)
    ho = ora.Hierarchy(rp, ci, va, np.ones(n), max_levels=max_levels, coarse_sweeps=7)
    zo = ho.vcycle(r)
    for precision, tol in (("fp64", ENTRY_FP64), ("fp32", ENTRY_FP32)):
        h = B.Hierarchy(rp, ci, va, precision=precision, max_levels=max_levels, coarse_sweeps=7)
        assert h.info()["nl"] == max_levels
        _close_entries(h.precond(r).cpu().numpy(), zo, tol)
        h.close()
