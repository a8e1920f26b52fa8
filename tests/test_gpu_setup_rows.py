"""Setup paths chosen by row length and density, against the oracle: rows of
more than 4 G entries in the matching and Galerkin kernels (a whole wave each),
and the sweep operator of a coarsest level too large for one workgroup's LDS
(doubling on the matrix cores, A dense or sparse)."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP64, B, _bits, _close_entries, _compare_hierarchy, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _spokes(n, degrees, base, seed):
    """A ring with `base` short chords a row, and hubs of the given degrees."""
    rng = np.random.default_rng(seed)
    r = [np.arange(n)]
    c = [(np.arange(n) + 1) % n]
    for k in range(base):
        r.append(np.arange(n))
        c.append((np.arange(n) + 2 + k) % n)
    for t, d in enumerate(degrees):
        hub = (t * n) // len(degrees)
        leaves = rng.choice(np.delete(np.arange(n), hub), d, replace=False)
        r.append(np.full(d, hub))
        c.append(leaves)
    r, c = np.concatenate(r), np.concatenate(c)
    key = np.unique(np.minimum(r, c) * n + np.maximum(r, c))
    lo, hi = key // n, key % n
    keep = lo != hi
    lo, hi = lo[keep], hi[keep]
    v = rng.uniform(0.1, 1.0, len(lo))
    v[::7] = 0.25  # some equal weights
    W = sp.coo_matrix((np.concatenate([-v, -v]), (np.concatenate([lo, hi]), np.concatenate([hi, lo]))), shape=(n, n)).tocsr()
    A = (W + sp.diags(-np.asarray(W.sum(axis=1)).ravel() + 0.1)).tocsr()
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data.copy()


# mean row length -> lanes per row G; degrees around 2 G (the cycle legs' mid
# rows), 4 G, the wave's slots (256) and 16 G, the bound of the long rows
ROWS = [(4, 0, (5, 6, 7, 11, 12, 13, 14, 30, 59, 60, 61, 62, 63, 64, 200)),
        (8, 1, (10, 11, 12, 13, 25, 26, 27, 28, 29, 60, 120, 121, 122, 123, 124, 125, 300)),
        (16, 5, (17, 18, 19, 20, 21, 50, 51, 52, 53, 54, 120, 200, 240, 241, 242, 243, 244, 245, 500)),
        (32, 10, (100, 105, 106, 107, 108, 200, 230, 234, 235, 236, 240, 400, 489, 490, 491, 492, 900))]


@pytest.mark.parametrize("G,base,degrees", ROWS)
def test_rows_around_the_lane_bounds(B, ora, G, base, degrees):  # noqa: F811
    n = 1500
    rp, ci, va = _spokes(n, degrees * 3, base, G)
    w = np.ones(n)
    say(f"rows around the bounds of G={G}: mean {np.diff(rp).mean():.1f} longest {np.diff(rp).max()}")
    c_ref = ora.weights(rp, ci, va, w)
    mate, c = B.match(rp, ci, va, w)
    assert np.array_equal(_bits(c.cpu().numpy()), _bits(c_ref))
    assert np.array_equal(mate.cpu().numpy(), ora.match(rp, ci, c_ref))
    for group in (0, G):
        h = B.Hierarchy(rp, ci, va, max_coarse=30, group=group)
        ho = ora.Hierarchy(rp, ci, va, w, max_coarse=30)
        _compare_hierarchy(h, ho)
        r = P.uniform_rhs(n, 3)
        _close_entries(h.precond(r).cpu().numpy(), ho.vcycle(r), ENTRY_FP64)
        h.close()


@pytest.mark.parametrize("n,degree", [(257, 120), (577, 30), (1025, 12), (1025, 400), (2048, 40)])
@pytest.mark.parametrize("sweeps", [1, 2, 3, 20, 23])
def test_sweep_operator_of_the_coarsest_level(B, ora, n, degree, sweeps):  # noqa: F811
    # one level: the cycle is the coarsest solve, applied as a dense operator.
    # Doubling rounds each entry a few dozen times more than the sweeps do, on
    # terms of the result's size: the entry bound of the folded operators
    rp, ci, va = P.random_spd(n, degree / n, n + degree)
    say(f"sweep operator n={n} nnz={len(ci)} sweeps={sweeps}")
    r = P.uniform_rhs(n, 5)
    zo = ora.Hierarchy(rp, ci, va, np.ones(n), max_coarse=n, coarse_sweeps=sweeps).vcycle(r)
    for check in (True, False):
        h = B.Hierarchy(rp, ci, va, max_coarse=n, coarse_sweeps=sweeps, check=check)
        _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64)
        h.close()
