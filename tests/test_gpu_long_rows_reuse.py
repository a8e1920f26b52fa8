"""Solves and cycles in turn on one handle whose finest level holds long (hub) rows.

The finest down leg takes the flexible-CG stop test and counts the arrivals of the
long rows' chunks in the same launch: the launch in which a solve ends must leave
the counters as it found them, so what a handle returns cannot depend on the solves
before.  All sums are taken in a fixed order: repeated calls agree bit for bit.
"""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP32, ENTRY_FP64, B, _bits, _close_entries, _fp32_allowance, _hubs, _two_hubs_paired, say  # noqa: F401,E501

pytestmark = pytest.mark.gpu


def _dense(n, seed):
    """Every row couples to every other one: all rows are long, in two chunks each
    (more chunk workgroups than are resident at once)."""
    rng = np.random.default_rng(seed)
    a = np.triu(-rng.uniform(0.1, 1.0, (n, n)), 1)
    a += a.T
    a[np.arange(n), np.arange(n)] = -a.sum(axis=1) * 1.02
    return (np.arange(n + 1, dtype=np.int32) * n, np.tile(np.arange(n, dtype=np.int32), n), a.ravel().copy())


CASES = {
    "dense 2100": lambda: _dense(2100, 1),
    "three hubs": lambda: _hubs(n_leaf=40000, hubs=(0, 17000, 40002), frac=0.5),
    "two hubs in one aggregate": _two_hubs_paired,
}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", list(CASES))
def test_solves_and_cycles_in_turn(B, ora, case, precision):  # noqa: F811
    rp, ci, va = CASES[case]()
    n = len(rp) - 1
    say(f"long rows, one handle: {case} {precision} n={n} longest={np.diff(rp).max()}")
    A = sp.csr_matrix((va, ci, rp), shape=(n, n))
    ho = ora.Hierarchy(rp, ci, va, np.ones(n), max_coarse=50)
    r, b1, b2 = (P.uniform_rhs(n, s) for s in (51, 52, 53))
    zo = ho.vcycle(r)
    its = [ho.solve(b, tol=1e-8)[1]["iters"] for b in (b1, b2)]
    for graph in (False, True):
        h = B.Hierarchy(rp, ci, va, max_coarse=50, precision=precision, graph=graph)
        assert h.info()["n"] == ho.sizes() and int(np.diff(rp).max()) > 1024
        z0 = h.precond(r).cpu().numpy()
        _close_entries(z0, zo, ENTRY_FP64 if precision == "fp64" else ENTRY_FP32)
        first = {}
        for turn in range(3):
            for k, b in enumerate((b1, b2)):
                x = h.solve(b, tol=1e-8).cpu().numpy()
                allow = 1 if precision == "fp64" else _fp32_allowance(its[k])
                assert abs(h.info()["iters"] - its[k]) <= allow, (h.info()["iters"], its[k])
                assert np.linalg.norm(b - A @ x) <= 1e-8 * np.linalg.norm(b)
                assert np.array_equal(_bits(x), _bits(first.setdefault(k, x))), "a solve differs from the first"
                z = h.precond(r).cpu().numpy()
                assert np.array_equal(_bits(z), _bits(z0)), "the cycle differs after a solve"
        h.close()
