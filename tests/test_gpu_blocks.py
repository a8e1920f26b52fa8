"""Sliced-ELL slices whose rows share offsets by blocks of 2 or 3 unknowns, in the
split legs and the flexible-CG product, against the oracle: the sums of a row are
taken in another order (its parts by wave), the bounds are those of one FP64 or
FP32 cycle and of the first flexible-CG iterates."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP32, ENTRY_FP64, B, _close_entries, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _nodes(m, B, drop, seed):
    """B unknowns on each node of an m^3 grid, coupled to the 27 neighbouring
    nodes by random blocks; a share `drop` of the couplings taken out (rows then
    hold a part of the shared list)."""
    rng = np.random.default_rng(seed)
    T = sp.diags([np.ones(m - 1), np.ones(m), np.ones(m - 1)], [-1, 0, 1])
    N = sp.triu(sp.kron(T, sp.kron(T, T)), 1).tocoo()
    keep = rng.uniform(size=N.nnz) >= drop
    r, c = N.row[keep], N.col[keep]
    n = B * m ** 3
    rows = (B * r[:, None, None] + np.arange(B)[:, None]).repeat(B, 2).ravel()
    cols = (B * c[:, None, None] + np.arange(B)[None, :]).repeat(B, 1).ravel()
    v = -rng.uniform(0.1, 1.0, len(rows))
    W = sp.coo_matrix((np.concatenate([v, v]), (np.concatenate([rows, cols]), np.concatenate([cols, rows]))),
                      shape=(n, n)).tocsr()
    A = (W + sp.diags(-np.asarray(W.sum(axis=1)).ravel() * 1.05)).tocsr()
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data.copy()


CASES = {"elasticity 17": lambda: P.elasticity3d(17, 4)[:3],
         "two unknowns": lambda: _nodes(23, 2, 0.0, 1), "two unknowns, holes": lambda: _nodes(25, 2, 0.1, 2),
         "three unknowns, holes": lambda: _nodes(19, 3, 0.05, 3)}


@pytest.mark.parametrize("name", list(CASES))
def test_block_uniform_slices(B, ora, name):  # noqa: F811
    rp, ci, va = CASES[name]()
    n = len(rp) - 1
    assert len(ci) >= 1 << 20, "the split legs need 2^20 entries"
    say(f"block-uniform slices: {name} n={n} nnz={len(ci)}")
    ho = ora.Hierarchy(rp, ci, va, np.ones(n))
    r = P.uniform_rhs(n, 3)
    zo = ho.vcycle(r)
    xo = ho.solve(r, tol=1e-30, itmax=3)[0]
    for precision, cyc, it in (("fp64", ENTRY_FP64, 1e-12), ("fp32", ENTRY_FP32, 1e-5)):
        h = B.Hierarchy(rp, ci, va, precision=precision, itmax=3)
        _close_entries(h.precond(r).cpu().numpy(), zo, cyc)
        _close_entries(h.solve(r, tol=1e-30, allow_maxit=True).cpu().numpy(), xo, it)
        h.close()
