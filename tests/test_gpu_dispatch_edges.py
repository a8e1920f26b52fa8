"""Both sides of the lines at which a path changes, against the oracle: the Suitor
matching in LDS (up to 4096 vertices, 2560 of rows of two to eight dozen entries), the coarsest sweeps by powers (where the square
is taken or refused by its lanes and entries), the down leg on the values of A D in FP64
(levels of 2^19 rows, values that are no float32), the flexible-CG stop test in the
fused down leg (aggregates of up to four rows) and the W-cycle's second result added
by the up leg.  Matchings bit for bit; cycles within the entry-wise bounds of one
cycle; repeated solves on one handle bit for bit."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP32, ENTRY_FP64, B, _bits, _close_entries, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _irregular(n, seed, equal, more=0):
    """A random graph Laplacian plus a small diagonal: rows of 2 to about 40 entries
    (and 2 `more`), a third of the weights (equal: all of them) the same."""
    rng = np.random.default_rng(seed)
    deg = np.minimum(rng.geometric(0.25, n), 30) + more
    lo = np.repeat(np.arange(n), deg)
    hi = rng.integers(0, n, len(lo))
    keep = lo != hi
    key = np.unique(np.minimum(lo, hi)[keep] * n + np.maximum(lo, hi)[keep])
    lo, hi = key // n, key % n
    v = rng.uniform(0.1, 1.0, len(lo))
    v[slice(None) if equal else slice(0, None, 3)] = 0.5
    W = sp.coo_matrix((np.concatenate([-v, -v]), (np.concatenate([lo, hi]), np.concatenate([hi, lo]))),
                      shape=(n, n)).tocsr()
    A = (W + sp.diags(np.full(n, 1.0) if equal else -np.asarray(W.sum(axis=1)).ravel() + 0.25)).tocsr()
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data.copy()


@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("n,more", [(2, 0), (1023, 0), (1024, 0), (1025, 0), (4095, 0), (4096, 0), (4097, 0),
                                    (1024, 20), (2559, 20), (2560, 20), (2561, 20), (4096, 60), (4097, 60)])
def test_suitor_on_small_graphs(B, ora, n, more, equal):  # noqa: F811
    rp, ci, va = _irregular(n, n, equal, more)
    assert {0: (0, 24), 20: (24, 96), 60: (96, 999)}[more][0] <= len(ci) / n < {0: (0, 24), 20: (24, 96), 60: (96, 999)}[more][1]
    w = np.ones(n)
    say(f"suitor n={n} nnz={len(ci)} equal={equal}")
    c_ref = ora.weights(rp, ci, va, w)
    for noalloc in (False, True):
        mate, c = B.match(rp, ci, va, w, noalloc=noalloc)
        assert np.array_equal(_bits(c.cpu().numpy()), _bits(c_ref))
        assert np.array_equal(mate.cpu().numpy(), ora.match(rp, ci, c_ref))


@pytest.mark.parametrize("shape", [(80, 80, 80), (81, 81, 80)])
def test_fp64_values_of_A_D(B, ora, shape):  # noqa: F811
    nx, ny, nz = shape
    rng = np.random.default_rng(nx + ny)
    kap = np.exp(rng.standard_normal((nz, ny, nx)))
    n = nx * ny * nz
    idx = np.arange(n).reshape(nz, ny, nx)
    rows, cols, vals, diag = [], [], [], np.full((nz, ny, nx), 0.01)
    for ax in range(3):
        a, b = [slice(None)] * 3, [slice(None)] * 3
        a[ax], b[ax] = slice(None, -1), slice(1, None)
        a, b = tuple(a), tuple(b)
        t = 2.0 * kap[a] * kap[b] / (kap[a] + kap[b])
        diag[a] += t
        diag[b] += t
        rows += [idx[a].ravel(), idx[b].ravel()]
        cols += [idx[b].ravel(), idx[a].ravel()]
        vals += [-t.ravel(), -t.ravel()]
    A = (sp.coo_matrix((np.concatenate(vals), (np.concatenate(rows), np.concatenate(cols))), shape=(n, n)) +
         sp.diags(diag.ravel())).tocsr()
    A.sort_indices()
    rp, ci, va = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data.copy()
    say(f"FP64 values of A D: n={n} (2^19 = {1 << 19})")
    r = P.uniform_rhs(n, 71)
    h = B.Hierarchy(rp, ci, va, min_ratio=2.0)
    ho = ora.Hierarchy(rp, ci, va, np.ones(n), min_ratio=2.0)
    assert h.info()["n"] == ho.sizes()
    _close_entries(h.precond(r).cpu().numpy(), ho.vcycle(r), ENTRY_FP64)
    h.close()


@pytest.mark.parametrize("sweeps", [1, 2, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_stop_test_on_a_reused_handle(B, ora, sweeps, precision):  # noqa: F811
    # finest levels on the fused down leg: aggregates of two and of four rows (the leg
    # takes the stop test) and of eight (a launch of its own)
    rp, ci, va = P.diffusion3d(24, 1.0, 3)[:3]
    n = len(rp) - 1
    say(f"stop test, one handle: sweeps={sweeps} {precision}")
    ho = ora.Hierarchy(rp, ci, va, np.ones(n), sweeps=sweeps, max_coarse=200)
    bs = [P.uniform_rhs(n, s) for s in (72, 73)]
    its = [ho.solve(b, tol=1e-9)[1]["iters"] for b in bs]
    A = sp.csr_matrix((va, ci, rp), shape=(n, n))
    for graph in (False, True):
        h = B.Hierarchy(rp, ci, va, sweeps=sweeps, max_coarse=200, precision=precision, graph=graph)
        first = {}
        for turn in range(2):
            for k, b in enumerate(bs):
                x = h.solve(b, tol=1e-9).cpu().numpy()
                got = h.info()["iters"]
                assert abs(got - its[k]) <= (1 if precision == "fp64" else max(2, its[k] // 20)), (got, its[k])
                assert np.linalg.norm(b - A @ x) <= 1e-9 * np.linalg.norm(b)
                x0, it0 = first.setdefault(k, (x, got))
                assert got == it0 and np.array_equal(_bits(x), _bits(x0))
            # an iteration limit ends the loop in the same place
            h5 = B.Hierarchy(rp, ci, va, sweeps=sweeps, max_coarse=200, precision=precision, graph=graph, itmax=5)
            h5.solve(bs[0], tol=1e-12, allow_maxit=True)
            assert h5.info()["iters"] == 5 and h5.info()["status"] == B.BCM_MAXIT
            h5.close()
        h.close()


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("matrix,levels", [("poisson", 3), ("poisson", 5), ("hubs", 3)])
def test_second_result_of_the_w_cycle(B, ora, matrix, levels, precision, fold):  # noqa: F811
    # the up leg of every level above the folded one adds the first result; hubs: in
    # its chunk and mid blocks too
    if matrix == "poisson":
        rp, ci, va = P.poisson3d(25, 23, 27)
    else:
        from test_gpu_parity import _hubs
        rp, ci, va = _hubs(n_leaf=20000, hubs=(0, 9000), frac=0.4)
    n = len(rp) - 1
    say(f"W-cycle: {matrix} n={n} levels={levels} {precision} fold={fold}")
    ho = ora.Hierarchy(rp, ci, va, np.ones(n), max_levels=levels, max_coarse=30, cycle="W")
    h = B.Hierarchy(rp, ci, va, max_levels=levels, max_coarse=30, cycle="W", precision=precision, fold=fold)
    assert h.info()["n"] == ho.sizes()
    for seed in (74, 75, 76):  # (the level's two result vectors change places from cycle to cycle)
        r = P.uniform_rhs(n, seed)
        _close_entries(h.precond(r).cpu().numpy(), ho.vcycle(r), ENTRY_FP64 if precision == "fp64" else ENTRY_FP32)
    h.close()


POWERS = {"65,536 rows of 32 lanes": lambda: P.poisson2d(256), "65,792 rows": lambda: P.poisson2d(256, 257),
          "64,000 rows, 1.5 M entries": lambda: P.poisson3d(40), "1.5 M entries of 110 a row": lambda: P.random_spd(13500, 11 / 13500, 2),
          "1.8 M entries of 110 a row": lambda: P.random_spd(16000, 11 / 16000, 2),
          "2.0 M entries of 400 a row": lambda: P.random_spd(5000, 21 / 5000, 2),
          "2.4 M entries of 400 a row": lambda: P.random_spd(6000, 21 / 6000, 2)}


@pytest.mark.parametrize("name", list(POWERS))
def test_sweeps_where_the_square_is_taken_or_refused(B, ora, name):  # noqa: F811
    rp, ci, va = POWERS[name]()[:3]
    n = len(rp) - 1
    say(f"powers: {name} n={n} nnz={len(ci)}")
    r = P.uniform_rhs(n, 77)
    zo = ora.Hierarchy(rp, ci, va, np.ones(n), max_levels=1).vcycle(r)
    h = B.Hierarchy(rp, ci, va, max_levels=1)
    _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64)
    h.close()


@pytest.mark.parametrize("n,degree", [(90, 60), (128, 120), (192, 60), (256, 25), (256, 250), (257, 60)])
@pytest.mark.parametrize("sweeps", [1, 2, 4, 7, 20])
def test_sweep_operator_of_small_dense_levels(B, ora, n, degree, sweeps):  # noqa: F811
    # unit vectors or doubling, by sweeps, rows and entries; matrices that no workgroup's
    # LDS holds
    rp, ci, va = P.random_spd(n, degree / n, n + degree)
    assert 16 * n + 12 * len(ci) + 4 * (n + 1) > 65536
    say(f"small sweep operator n={n} nnz={len(ci)} sweeps={sweeps}")
    r = P.uniform_rhs(n, 78)
    zo = ora.Hierarchy(rp, ci, va, np.ones(n), max_coarse=n, coarse_sweeps=sweeps).vcycle(r)
    for check in (True, False):
        h = B.Hierarchy(rp, ci, va, max_coarse=n, coarse_sweeps=sweeps, check=check)
        _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64)
        h.close()
