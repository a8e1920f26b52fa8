"""Device memory of the setup's optional forms (the coarsest sweeps by powers, star
levels as one operator): what is tried and not taken is given back, and a form that cannot be allocated
leaves the levels' own kernels, with the same results."""
import numpy as np
import pytest

from paper_1810_04221_amd import problems as P
from test_gpu_parity import ENTRY_FP32, ENTRY_FP64, B, _close_entries, say  # noqa: F401
from test_gpu_star import _star

pytestmark = pytest.mark.gpu


@pytest.fixture
def meter(B, monkeypatch):  # noqa: F811
    """The library's allocator with a count of what it holds and, when set, a limit."""
    base = B._TorchAllocator

    class Meter(base):
        limit = None

        def __init__(self, device, stream):
            super().__init__(device, stream)
            self.live = self.peak = 0
            take, give = self.alloc, self.dealloc

            def alloc(size, ctx):
                if Meter.limit is not None and self.live + size > Meter.limit:
                    return None
                p = take(size, ctx)
                if p:
                    self.live += size
                    self.peak = max(self.peak, self.live)
                return p

            def dealloc(ptr, size, ctx):
                self.live -= size
                give(ptr, size, ctx)

            self.alloc, self.dealloc = B.ALLOC_FN(alloc), B.DEALLOC_FN(dealloc)
            self.keep = take, give

    monkeypatch.setattr(B, "_TorchAllocator", Meter)
    return Meter


def test_refused_powers_hold_no_memory(B, meter):  # noqa: F811
    # one level of 125,000 rows: the square has too many entries.  An odd number of
    # sweeps never tries it: the two handles hold the same memory
    rp, ci, va = P.poisson3d(50)
    say("refused powers: poisson3d 50^3, one level")
    held, peak = [], []
    for sweeps in (21, 20):
        h = B.Hierarchy(rp, ci, va, max_levels=1, coarse_sweeps=sweeps)
        held.append(h._alloc.live)
        peak.append(h._alloc.peak)
        h.close()
        assert h._alloc.live == 0
    assert held[0] == held[1] and peak[0] == peak[1], (held, peak)


def test_powers_without_memory_for_them(B, ora, meter):  # noqa: F811
    # 62,500 rows, whose square is taken: with just the memory of a setup that does
    # not try it, the sweeps stay one by one
    rp, ci, va = P.poisson2d(250)
    n = len(rp) - 1
    say(f"powers without memory: poisson2d 250^2 n={n}, one level")
    r = P.uniform_rhs(n, 8)
    h = B.Hierarchy(rp, ci, va, max_levels=1, coarse_sweeps=21)
    bare, limit = h._alloc.live, h._alloc.peak
    h.close()
    zo = ora.Hierarchy(rp, ci, va, np.ones(n), max_levels=1, coarse_sweeps=20).vcycle(r)
    for lim in (None, limit):
        meter.limit = lim
        h = B.Hierarchy(rp, ci, va, max_levels=1, coarse_sweeps=20)
        assert (h._alloc.live == bare) == (lim is not None)
        _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64)
        h.close()


@pytest.mark.parametrize("sweeps", [2, 4, 6])
def test_few_sweeps_form_no_powers(B, meter, sweeps):  # noqa: F811
    # a cycle of so few sweeps does not repay the powers that a setup would form
    rp, ci, va = P.poisson2d(250)
    say(f"few sweeps: poisson2d 250^2, {sweeps} sweeps")
    live = []
    for s in (sweeps + 1, sweeps, 8):
        h = B.Hierarchy(rp, ci, va, max_levels=1, coarse_sweeps=s)
        live.append(h._alloc.live)
        h.close()
    assert live[0] == live[1] < live[2], live


@pytest.mark.parametrize("n,levels,bare", [(160000, 12, dict(fold=False)), (300000, 1, dict(coarse_sweeps=33))])
def test_chain_without_memory_for_it(B, ora, meter, n, levels, bare):  # noqa: F811
    # a chain of stars, and a coarsest star alone: with just the memory of a setup that
    # does not form their operator (33 sweeps are beyond it) the levels keep their own
    # kernels
    rp, ci, va = _star(n, 5, n)
    say(f"chain without memory: n={n} levels={levels}")
    h = B.Hierarchy(rp, ci, va, max_coarse=20, max_levels=levels, **bare)
    live, limit = h._alloc.live, h._alloc.peak
    h.close()
    r = P.uniform_rhs(n, 9)
    zo = ora.Hierarchy(rp, ci, va, np.ones(n), max_coarse=20, max_levels=levels).vcycle(r)
    for lim in (None, limit):
        meter.limit = lim
        h = B.Hierarchy(rp, ci, va, max_coarse=20, max_levels=levels)
        if lim is not None:
            assert h._alloc.live == live
        _close_entries(h.precond(r).cpu().numpy(), zo, ENTRY_FP64)
        h.close()


@pytest.mark.parametrize("case,bare", [("diffusion fp64", dict(coarse_sweeps=21)), ("diffusion fp32", dict(coarse_sweeps=21)),
                                       ("star", dict(fold=False)), ("dense W", None)])
def test_setup_between_the_bare_and_the_full_memory(B, ora, meter, case, bare):  # noqa: F811
    # whatever the optional forms have taken before the memory ends: a setup that has
    # room for the levels' own kernels succeeds, with the same cycle
    rp, ci, va, kw = {
        "diffusion fp64": lambda: P.diffusion3d(84, 1.0, 3)[:3] + (dict(min_ratio=2.0),),
        "diffusion fp32": lambda: P.diffusion3d(84, 1.0, 3)[:3] + (dict(min_ratio=2.0, precision="fp32"),),
        "star": lambda: _star(160000, 5, 1) + (dict(max_levels=12, max_coarse=20),),
        "dense W": lambda: P.poisson2d(89)[:3] + (dict(max_levels=2, cycle="W"),)}[case]()
    n = len(rp) - 1
    say(f"setup between the bare and the full memory: {case} n={n}")
    r = P.uniform_rhs(n, 10)
    h = B.Hierarchy(rp, ci, va, **kw)
    full, z0, sizes = h._alloc.peak, h.precond(r).cpu().numpy(), h.info()["n"]
    h.close()
    if bare is not None:
        h = B.Hierarchy(rp, ci, va, **{**kw, **bare})
        low = h._alloc.peak
        h.close()
    else:  # without the three arrays of the doubling's scratch
        low = full - 3 * 8 * sizes[-1] ** 2
    assert low < full
    for k in range(9):
        meter.limit = low + (full - low) * k // 8
        h = B.Hierarchy(rp, ci, va, **kw)
        assert h.info()["n"] == sizes
        _close_entries(h.precond(r).cpu().numpy(), z0, ENTRY_FP32 if kw.get("precision") == "fp32" else ENTRY_FP64)
        x = h.solve(r, tol=1e-8)
        assert h.info()["relres"] <= 1e-8 and bool(x.isfinite().all())
        h.close()


def test_unsymmetric_star_holds_no_trial_levels(B, meter):  # noqa: F811
    # a star's pattern with one entry that differs from its transposed one by an ulp, not
    # checked: the general sweeps take every level, and what the star's sweeps had
    # allocated for it is given back
    n = 20000
    rp, ci, va = _star(n, 5, 7)
    say(f"unsymmetric star n={n}")
    live = []
    for odd in (False, True):
        v = va.copy()
        if odd:
            q = rp[n // 2 + 1] - 2  # row n / 2: its hub entry
            assert ci[q] == 5
            v[q] = np.nextafter(v[q], 0.0)
        h = B.Hierarchy(rp, ci, v, max_coarse=20, check=False, fold=False)
        assert h.info()["nl"] == 40
        live.append(h._alloc.live)
        h.close()
    assert live[1] <= live[0] + (64 << 20), live
