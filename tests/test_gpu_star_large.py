"""Star levels of so many rows that the sums over their leaves are finished by a
launch of their own, on both sides of that bound (20 chunks of 4096 rows), against
the oracle: a coarsest star alone and chains of a few levels.  The map is the
oracle's level-by-level cycle in another order; bounds as for the smaller stars."""
import numpy as np
import pytest

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP32, ENTRY_FP64, B, _close_entries, say  # noqa: F401
from test_gpu_star import _star

pytestmark = pytest.mark.gpu

FEW = 20 * 4096


@pytest.mark.parametrize("n,hub,levels,cycle", [(FEW, 7, 1, "V"), (FEW + 1, FEW, 1, "V"), (FEW + 5, 0, 4, "V"),
                                                (200003, 100000, 6, "V"), (FEW + 9, 3, 3, "W")])
def test_star_of_many_chunks(B, ora, n, hub, levels, cycle):  # noqa: F811
    rp, ci, va = _star(n, hub, n)
    w = np.ones(n)
    say(f"large star n={n} hub={hub} levels={levels} {cycle}")
    ho = ora.Hierarchy(rp, ci, va, w, max_coarse=20, max_levels=levels, cycle=cycle)
    r, b = P.uniform_rhs(n, 61), P.uniform_rhs(n, 62)
    zo, io = ho.vcycle(r), ho.solve(b, tol=1e-9)[1]
    for precision in ("fp64", "fp32"):
        h = B.Hierarchy(rp, ci, va, w, max_coarse=20, max_levels=levels, precision=precision, cycle=cycle)
        assert h.info()["n"] == ho.sizes()
        _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64 if precision == "fp64" else ENTRY_FP32)
        h.solve(b, tol=1e-9)
        assert abs(h.info()["iters"] - io["iters"]) <= (1 if precision == "fp64" else 2)
        h.close()
