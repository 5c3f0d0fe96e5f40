"""The coarsest-level solves at the sizes where their paths change: one wave
with one and with two cells a lane (up to 64 and 128 cells), then the group of
ceil(N / 128) waves up to 1024 cells, against the dense minimum-norm solution.
The grids have odd sides or an explicit level count, so the whole solve is the
coarsest one."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GRIDS = [((5, 3), (False, False)), ((8, 8), (True, True)), ((13, 5), (False, True)),
         ((16, 8), (False, False)), ((43, 3), (False, False)), ((11, 7, 5), (False, False, False)),
         ((9, 7, 11), (True, True, True)), ((16, 8, 8), (False, True, False)),
         ((32, 16), (False, False)), ((27, 19), (True, False)), ((32, 32), (False, False))]


def _dense(n, per, L):
    """-A of the coefficient-weighted stencil, face by face."""
    d, N = len(n), int(np.prod(n))
    idx = np.arange(N).reshape(tuple(reversed(n)))
    M = np.zeros((N, N))
    for i in range(d):
        ax = d - 1 - i
        lo = np.roll(idx, 1, ax)
        for c, q, w in zip(idx.ravel(), lo.ravel(), L[i].ravel()):
            if c != q:
                M[c, c] += w
                M[q, q] += w
                M[c, q] -= w
                M[q, c] -= w
    return M


def _problem(n, per, seed):
    rng = np.random.default_rng(seed)
    d = len(n)
    L = rng.uniform(0.5, 1.0, (d,) + tuple(reversed(n)))
    for i in range(d):
        if not per[i]:
            L[(i,) + tuple(slice(None) if a != d - 1 - i else 0 for a in range(d))] = 0.0
    b = rng.standard_normal(tuple(reversed(n)))
    return L, b - b.mean()


def _dev(a, n, dtype):
    shape = a.shape[:-len(n)] + (1,) * (3 - len(n)) + a.shape[-len(n):]
    return torch.from_numpy(a.reshape(shape).copy()).to(dtype).cuda().contiguous()


@pytest.mark.parametrize("prec", ["fp64", "fp64-cg", "fp32"])
@pytest.mark.parametrize("n,per", GRIDS, ids=["x".join(map(str, g[0])) for g in GRIDS])
def test_one_level_solve_is_the_minimum_norm_solution(n, per, prec, monkeypatch):
    """fp64 takes the level's inverse up to 512 cells, fp64-cg the iteration."""
    import paper_2304_08159_amd as wl
    if prec == "fp64-cg":
        monkeypatch.setenv("WL_DIRECT_COARSE", "0")
        prec = "fp64"
    dtype = torch.float64 if prec == "fp64" else torch.float32
    L, b = _problem(n, per, 3)
    M = _dense(n, per, L)
    ev = np.linalg.eigvalsh(M)
    kappa = ev[-1] / ev[1]                      # ev[0] = 0: the constant
    ref = np.linalg.lstsq(M, -b.ravel(), rcond=1e-13)[0]
    ps = wl.Poisson(n, per, prec=wl.WL_FP64 if prec == "fp64" else wl.WL_FP32, levels=1)
    x = torch.zeros(ps.shape, dtype=dtype, device="cuda")
    ps.solve(_dev(L, n, dtype), x, _dev(b, n, dtype), tol=0.0, max_vcycles=1,
             allow_not_converged=True)
    got = x.double().cpu().numpy().ravel()
    got = got - got.mean()
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    # the iteration's residual tolerance (1e-10, 1e-6 in FP32) times the
    # condition number, plus the FP32 rounding of coefficients, b and x
    tol = (1e-10 if prec == "fp64" else 1e-6 + 4 * 2.0 ** -24) * kappa
    print(n, prec, "relative error", err, "bound", tol, flush=True)
    assert err <= tol


@pytest.mark.parametrize("n,per", [GRIDS[2], GRIDS[4], GRIDS[5], GRIDS[6]],
                         ids=["13x5", "43x3", "11x7x5", "9x7x11"])
def test_batched_one_level_solve_is_the_minimum_norm_solution(n, per):
    import paper_2304_08159_amd as wl
    L, b = _problem(n, per, 4)
    M = _dense(n, per, L)
    ev = np.linalg.eigvalsh(M)
    ref = np.linalg.lstsq(M, -b.ravel(), rcond=1e-13)[0]
    Ld, bd = _dev(L, n, torch.float64), _dev(b, n, torch.float64)
    x = torch.zeros_like(bd)
    out = wl.poisson_batch_solve([dict(n=n, periodic=per, coeffs=Ld, x=x, b=bd, tol=1e-9)])
    assert out[0][0] == 0 and out[0][1] <= 2
    got = x.cpu().numpy().ravel()
    got = got - got.mean()
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert err <= 1e-9 * ev[-1] / ev[1]
