"""The batched runs' momentum at sizes where the outermost two layers meet or
leave a single inner row, with walls, periodic directions and both: one step
from a random state against the FP64 oracle.  No body, so velocity and the
pressure in the operator's energy norm hold to 1e-5: some 100 FP32 roundings
(6e-8) of fields of order one."""

import math

import numpy as np
import pytest

from oracle import poisson as P
from oracle import step as S
from tests.gpu_util import mean_free, to_device, to_oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [((4, 8), (3, 3)), ((5, 7), (3, 0)), ((6, 16), (0, 3)), ((16, 4), (3, 3)), ((5, 5), (0, 0)),
         ((4, 5, 6), (3, 3, 3)), ((8, 4, 7), (0, 3, 3)), ((6, 6, 5), (3, 0, 0)),
         ((9, 5, 8), (0, 0, 3))]


@pytest.mark.parametrize("n,bc", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_one_step_where_layers_meet(n, bc):
    import paper_2304_08159_amd as wl
    d = len(n)
    rng = np.random.default_rng(11)
    comps = [rng.uniform(-1.0, 1.0, n).astype(np.float32).astype(np.float64) for _ in range(d)]
    for i in range(d):
        if bc[i] != 0:
            idx = [slice(None)] * d
            idx[i] = 0
            comps[i][tuple(idx)] = 0.0
    U, nu = (0.0,) * d, 0.05
    u = torch.stack([to_device(a, d, torch, torch.float32) for a in comps]).contiguous()
    p = torch.zeros(tuple(reversed(list(n) + [1] * (3 - d))), dtype=torch.float64, device="cuda")
    st, vc, t, dt = wl.ns_batch_run([dict(n=n, bc_lo=list(bc), bc_hi=list(bc), U=U, nu=nu, body=None,
                                          tol=1e-9, max_vcycles=200, steps=1, u=u, uout=None,
                                          p=p)])[0]
    assert st == 0
    osim = S.Sim(n, list(bc), list(bc), U, nu, body=None, tol=1e-12, stop_rule="relative",
                 max_vcycles=300)
    osim.u, osim.uout, osim.p = comps, None, np.zeros(n)
    osim.step(dt=dt)
    ug = [to_oracle(u[i], d) for i in range(d)]
    eu = math.sqrt(sum(np.sum((a - b) ** 2) for a, b in zip(ug, osim.u)) /
                   sum(np.sum(b ** 2) for b in osim.u))
    act = osim.h.active[0]
    pg, po = mean_free(to_oracle(p, d), act), mean_free(osim.p, act)
    per, e = [b == 0 for b in bc], pg - po
    ea = math.sqrt(abs(np.sum(e * P.apply_A(osim.L, e, per))) /
                   abs(np.sum(po * P.apply_A(osim.L, po, per))))
    print(n, bc, f"dt={dt:.4f} vc={vc} err_u={eu:.2e} err_p={ea:.2e}", flush=True)
    assert eu <= 1e-5 and ea <= 1e-5
