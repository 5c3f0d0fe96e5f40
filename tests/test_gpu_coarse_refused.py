"""Coarsest levels that have room for an inverse but are solved by the
iteration: no inverse attempted, or one refused because a row of it did not
converge."""

import time

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _solver(n, seed=1):
    """A one-level FP64 solver on a closed box, unit coefficients, a mean-free
    right-hand side."""
    import paper_2304_08159_amd as wl
    d = len(n)
    ps = wl.Poisson(n, (False,) * d, prec=wl.WL_FP64, levels=1)
    L = torch.ones((d,) + ps.shape, dtype=torch.float64, device="cuda")
    for i in range(d):
        L[i].select(2 - i, 0).zero_()
    g = torch.Generator().manual_seed(seed)
    b = torch.randn(ps.shape, generator=g, dtype=torch.float64).cuda()
    return ps, L, b - b.mean()


def _solve(ps, L, b):
    x = torch.zeros_like(b)
    ps.solve(L, x, b, tol=0.0, max_vcycles=1, allow_not_converged=True)
    return x


def _time(ps, L, b, reps=30):
    x = torch.zeros_like(b)
    ps.solve(L, x, b, tol=0.0, max_vcycles=1, allow_not_converged=True)
    best = 1e9
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(reps):
            x.zero_()
            ps.solve(None, x, b, tol=0.0, max_vcycles=1, allow_not_converged=True)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / reps)
    return best * 1e6


def test_iteration_without_an_inverse_runs_at_its_own_workgroup(monkeypatch):
    monkeypatch.setenv("WL_DIRECT_COARSE", "0")
    # 513 cells have no room for an inverse and take the iteration's workgroup;
    # three cells fewer are the same problem with room for one
    beyond, within = _time(*_solver((171, 3))), _time(*_solver((170, 3)))
    print("513 cells", round(beyond, 1), "us, 510 cells", round(within, 1), "us", flush=True)
    assert within <= 1.05 * beyond


def test_rows_that_are_no_numbers_are_refused():
    """Coefficients of 1e-310: a unit row divides by them and ends in NaN.  The
    iteration on a right-hand side of 1e-155 finds no descent (its products
    underflow) and leaves the zero correction."""
    ps, L, b = _solver((12, 11))
    x = _solve(ps, 1e-310 * L, 1e-155 * b)
    assert bool(torch.isfinite(x).all())
