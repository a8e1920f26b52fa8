"""Star levels on the GPU against the oracle: the one-launch sweeps of the setup
(bit-exact hierarchy) and the chain operator of the V-cycle.

The chain operator is the same linear map as the oracle's level-by-level cycle,
its sums taken in another order: one ulp-size error per operation on terms no
larger than the result's scale, so the entry-wise bounds of the folded
operators hold (1e-11 in FP64, 1e-4 in the FP32 cycle, whose input and output
vectors of the chain are float32).
"""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP32, ENTRY_FP64, B, _close_entries, _compare_hierarchy, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _star(n, hub, seed, equal=False):
    """One hub coupled to every other row; equal: equal weights (ties by index)."""
    rng = np.random.default_rng(seed)
    a = np.full(n, -0.5) if equal else -rng.uniform(0.1, 1.0, n)
    leaves = np.delete(np.arange(n), hub)
    d = np.full(n, 1.0) if equal else np.abs(a) * rng.uniform(1.0, 2.0, n)
    d[hub] = 1.1 * np.abs(a[leaves]).sum()
    rows = np.concatenate([leaves, np.full(n - 1, hub), np.arange(n)])
    cols = np.concatenate([np.full(n - 1, hub), leaves, np.arange(n)])
    A = sp.csr_matrix((np.concatenate([a[leaves], a[leaves], d]), (rows, cols)), shape=(n, n))
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data.copy()


CASES = [
    # rows, hub row, sweeps per level, levels, equal weights, signed w
    (70, 0, 2, 40, False, False),
    (257, 256, 1, 40, False, True),
    (1100, 500, 2, 3, True, False),
    (2113, 0, 3, 40, False, True),
    (4096 + 5, 4100, 4, 9, False, False),
    (9001, 4444, 2, 40, True, True),
]


@pytest.mark.parametrize("n,hub,sweeps,levels,equal,signed", CASES)
def test_star_chain(B, ora, n, hub, sweeps, levels, equal, signed):  # noqa: F811
    rp, ci, va = _star(n, hub, n)
    if equal:
        rp, ci, va = _star(n, hub, n, equal=True)
    w = np.random.default_rng(n + 1).uniform(0.5, 2.0, n) if signed else np.ones(n)
    if signed:
        w[::3] *= -1.0
    say(f"star chain n={n} hub={hub} sweeps={sweeps} levels={levels} equal={equal} signed={signed}")
    ho = ora.Hierarchy(rp, ci, va, w, max_coarse=20, sweeps=sweeps, max_levels=levels)
    r = P.uniform_rhs(n, 31)
    zo = ho.vcycle(r)
    for precision, fold in (("fp64", True), ("fp64", False), ("fp32", True)):
        h = B.Hierarchy(rp, ci, va, w, max_coarse=20, sweeps=sweeps, max_levels=levels, precision=precision, fold=fold)
        _compare_hierarchy(h, ho)
        if n > 64:
            assert h.info()["long_rows"] == sum(m > 64 for m in ho.sizes())
        _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64 if precision == "fp64" else ENTRY_FP32)
        h.close()


@pytest.mark.parametrize("nx,sigma,max_coarse", [(20, 2.0, 100), (32, 1.0, 200), (48, 1.0, 0)])
def test_stalled_hierarchy_chain(B, ora, nx, sigma, max_coarse):  # noqa: F811
    # diffusion whose coarsening stalls: general levels, then stars (on the small
    # grids the chain enters the folded operator in its dense form)
    rp, ci, va = P.diffusion3d(nx, sigma, 5)
    n = nx ** 3
    say(f"stalled hierarchy {nx}^3 sigma={sigma}")
    ho = ora.Hierarchy(rp, ci, va, np.ones(n), max_coarse=max_coarse or None)
    r, b = P.uniform_rhs(n, 33), P.uniform_rhs(n, 34)
    zo = ho.vcycle(r)
    _, io = ho.solve(b, tol=1e-8)
    for precision in ("fp64", "fp32"):
        h = B.Hierarchy(rp, ci, va, max_coarse=max_coarse, precision=precision)
        _compare_hierarchy(h, ho)
        _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64 if precision == "fp64" else ENTRY_FP32)
        x = h.solve(b, tol=1e-8).cpu().numpy()
        A = sp.csr_matrix((va, ci, rp), shape=(n, n))
        assert np.linalg.norm(b - A @ x) <= 1e-8 * np.linalg.norm(b)
        assert abs(h.info()["iters"] - io["iters"]) <= (1 if precision == "fp64" else max(2, io["iters"] // 20))
        h.close()
