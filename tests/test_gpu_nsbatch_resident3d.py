"""Batched 3D runs whose pressure solves are resident in one workgroup (512
threads, at most 512 lateral columns and 16 rows a thread): steps replayed by the
FP64 oracle at the column and row limits, with a last segment shorter than the
others, with inflow / outflow past a sphere, walls and periodic directions; and
the kernel that served them."""

import math

import numpy as np
import pytest

from oracle import momentum as M
from oracle import poisson as P
from oracle import step as S
from tests.gpu_util import mean_free, plane_to_oracle, rel_l2, to_device, to_oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FLOW = dict(bc_lo=[1, 3, 3], bc_hi=[2, 3, 3], U=(1.0, 0.0, 0.0), nu=0.06)
CASES = {
    # 512 columns of 16 rows: both limits
    "32x16x16 sphere": dict(FLOW, n=(32, 16, 16), body=dict(centre=(9.0, 8.2, 7.9), radius=2.5)),
    # two segments of 8 rows
    "16x16x16 sphere": dict(FLOW, n=(16, 16, 16), body=dict(centre=(5.0, 8.2, 7.9), radius=2.0)),
    # four segments, the last of two rows; a periodic walk direction
    "16x8x20 sphere": dict(FLOW, n=(16, 8, 20), bc_lo=[1, 3, 0], bc_hi=[2, 3, 0],
                           body=dict(centre=(5.0, 4.1, 9.9), radius=1.5)),
    # one segment of 12 rows for 384 of the threads; no body
    "24x16x12 walls": dict(n=(24, 16, 12), bc_lo=[3, 0, 3], bc_hi=[3, 0, 3], U=(0.0,) * 3, nu=0.05,
                           body=None),
    "16x16x16 periodic": dict(n=(16, 16, 16), bc_lo=[0] * 3, bc_hi=[0] * 3, U=(0.0,) * 3, nu=0.05,
                              body=None),
    # 64 columns, eight segments of two rows
    "8x8x16 walls": dict(n=(8, 8, 16), bc_lo=[3] * 3, bc_hi=[3] * 3, U=(0.0,) * 3, nu=0.05,
                         body=None),
}


def _request(cfg, steps):
    n, d = cfg["n"], 3
    rng = np.random.default_rng(5)
    # a random disturbance (of order one without a stream), boundary faces at their value
    amp = 1.0 if cfg["body"] is None else 0.05
    comps = [cfg["U"][i] + amp * rng.uniform(-1.0, 1.0, n) for i in range(d)]
    for i in range(d):
        if cfg["bc_lo"][i] != 0:
            idx = [slice(None)] * d
            idx[i] = 0
            comps[i][tuple(idx)] = cfg["U"][i] if cfg["bc_lo"][i] == 1 else 0.0
    u = torch.stack([to_device(a, d, torch, torch.float32) for a in comps]).contiguous()
    p = torch.zeros(tuple(reversed(n)), dtype=torch.float64, device="cuda")
    uout = torch.full((n[2], n[1]), cfg["U"][0], device="cuda") if cfg["bc_hi"][0] == 2 else None
    return dict(n=n, bc_lo=cfg["bc_lo"], bc_hi=cfg["bc_hi"], U=cfg["U"], nu=cfg["nu"],
                body=cfg["body"], tol=1e-9, max_vcycles=200, steps=steps, u=u, uout=uout, p=p)


@pytest.mark.parametrize("name", list(CASES))
def test_steps_replay_against_the_oracle(name):
    """As the general path's replay: velocity and outflow plane to 1e-5 (about
    100 FP32 roundings of fields of order one), pressure to 1e-5 in the
    operator's energy norm."""
    import paper_2304_08159_amd as wl
    cfg, d = CASES[name], 3
    r = _request(cfg, 1)
    u, uout, p = r["u"], r["uout"], r["p"]
    osim = S.Sim(cfg["n"], cfg["bc_lo"], cfg["bc_hi"], cfg["U"], cfg["nu"], body=cfg["body"],
                 tol=1e-12, stop_rule="relative", max_vcycles=300)
    for step in range(3):
        un = [to_oracle(u[i], d) for i in range(d)]
        uo = plane_to_oracle(uout, d) if uout is not None else None
        pn = to_oracle(p, d)
        st, vc, t, dt = wl.ns_batch_run([r])[0]
        assert st == 0
        dt_o = M.cfl_dt(un, uo, cfg["bc_lo"], cfg["bc_hi"], cfg["U"], cfg["nu"], 0.5)
        osim.u, osim.uout, osim.p = un, uo, pn
        osim.step(dt=dt)
        ug = [to_oracle(u[i], d) for i in range(d)]
        eu = math.sqrt(sum(np.sum((a - b) ** 2) for a, b in zip(ug, osim.u)) /
                       sum(np.sum(b ** 2) for b in osim.u))
        act = osim.h.active[0]
        pg, po = mean_free(to_oracle(p, d), act), mean_free(osim.p, act)
        per, e = [b == 0 for b in cfg["bc_lo"]], pg - po
        ea = math.sqrt(abs(np.sum(e * P.apply_A(osim.L, e, per))) /
                       abs(np.sum(po * P.apply_A(osim.L, po, per))))
        eo = rel_l2(plane_to_oracle(uout, d), osim.uout) if uout is not None else 0.0
        print(f"{name} step {step}: dt={dt:.5f} (oracle {dt_o:.5f}) vc={vc} err_u={eu:.2e} "
              f"err_p={ea:.2e} err_uout={eo:.2e}", flush=True)
        assert abs(dt - dt_o) <= 1e-6 * dt_o
        assert eu <= 1e-5 and eo <= 1e-5 and ea <= 1e-5


@pytest.mark.parametrize("name", list(CASES))
def test_several_steps_in_one_call_equal_single_ones(name):
    """The class words and staged coefficients outlive the steps of a run: four
    steps in one call have the bits of four calls."""
    import paper_2304_08159_amd as wl
    a, b = _request(CASES[name], 4), _request(CASES[name], 1)
    assert wl.ns_batch_run([a])[0][0] == 0
    for _ in range(4):
        assert wl.ns_batch_run([b])[0][0] == 0
    for key in ("u", "p", "uout"):
        if a[key] is not None:
            assert torch.equal(a[key], b[key]), key


def test_these_runs_take_the_resident_3d_kernel():
    import paper_2304_08159_amd as wl
    reqs = [_request(c, 1) for c in CASES.values()]
    wl.ns_batch_run(reqs)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        wl.ns_batch_run(reqs)
        torch.cuda.synchronize()
    names = [e.key for e in prof.key_averages() if "k_ns_batch" in e.key]
    print(names, flush=True)
    if not names:
        pytest.skip("no kernel was traced here")
    assert len(names) == 1 and "k_ns_batch<2>" in names[0]
