"""The coarsest level's sweeps by powers of the sweep matrix against the oracle's
sweeps: the same polynomial in another order (each entry of a power is a sum of
at most 4096 products, a few ulp of the result's scale per application), so the
entry-wise bounds of the folded operators hold."""
import numpy as np
import pytest

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP32, ENTRY_FP64, B, _close_entries, say  # noqa: F401

pytestmark = pytest.mark.gpu


CASES = [
    # matrix, sweeps: M^4 and M^2 steps, one step alone, none (odd)
    ("poisson2d 61x47", lambda: P.poisson2d(61, 47), (20, 4, 2, 6, 18, 5)),
    ("poisson3d 17x13x11", lambda: P.poisson3d(17, 13, 11), (20, 8, 2)),
    ("random 2500", lambda: P.random_spd(2500, 4e-3, 3), (20, 6, 3)),    # M^4 nearly full: M^2
    ("random 2100 dense", lambda: P.random_spd(2100, 4e-2, 4), (20,)),   # too many products: sweeps
    ("elasticity 9", lambda: P.elasticity3d(9, 4)[:3], (20, 4)),
]


@pytest.mark.parametrize("name,make,sweeps", CASES, ids=[c[0] for c in CASES])
def test_coarsest_sweeps_by_powers(B, ora, name, make, sweeps):  # noqa: F811
    rp, ci, va = make()
    n = len(rp) - 1
    r = P.uniform_rhs(n, 7)
    for s in sweeps:
        for levels in (1, 2):  # the coarsest level alone (float64 vectors), and below one level
            say(f"powers {name} n={n} sweeps={s} levels={levels}")
            w = np.ones(n)
            if levels == 1:
                ho = ora.Hierarchy(rp, ci, va, w, max_coarse=n, coarse_sweeps=s)
            else:
                ho = ora.Hierarchy(rp, ci, va, w, max_levels=2, max_coarse=10, coarse_sweeps=s, sweeps=1)
            zo = ho.vcycle(r)
            for precision in ("fp64", "fp32") if levels == 2 else ("fp64",):
                h = B.Hierarchy(rp, ci, va, max_levels=levels, max_coarse=10, coarse_sweeps=s, sweeps=1,
                                precision=precision)
                assert h.info()["n"] == ho.sizes()
                _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64 if precision == "fp64" else ENTRY_FP32)
                h.close()
