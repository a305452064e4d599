"""LPA right-hand sides with masses in no panel of the radial sums: above them (late in
a flow), below them, and in a context whose budget cannot spare the table; with few
and many such points per wave, and a radial rule too wide
for the expansion above the panels.  Against the oracle, and the time within four
times that of a flow inside the panels."""
import numpy as np
import pytest

import oracle
from paper_2607_24908_amd import frg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EXP, LIT = frg.FRG_REG_EXP, frg.FRG_REG_LITIM
BUDGETS = {"table": 0, "no table": 1 << 20}


def dev(a):
    return torch.tensor(a, dtype=torch.float64, device="cuda")


def check(ctxs, reg, n_r, N, U, t=0.0, q_max=6.0):
    n = U.size
    want, wj, _ = oracle.lpa_rhs(3, N, reg, n_r, q_max, np.exp(t), 0.5, U, allow_domain=True)
    ok, wj = np.isfinite(want), np.asarray(wj).ravel()
    jk = np.tile(ok, 7)  # of a point outside the domain every band is NaN
    assert ok.any()
    lpa = frg.make_lpa(d=3, N=N, reg=reg, n_radial=n_r, q_max_over_k=q_max, n_grid=n)
    for ctx in ctxs:
        dU, J = dev(np.full(n, np.nan)), dev(np.full(7 * n, np.nan))
        frg.frg_flow_rhs(ctx, lpa, t, dev(U), dU, J)
        frg.frg_stream_status(ctx, allow_domain=True)
        got = dU.cpu().numpy()
        assert np.array_equal(ok, np.isfinite(got))
        assert np.abs(got[ok] / want[ok] - 1.0).max() < 1e-12
        assert np.abs(J.cpu().numpy()[jk] - wj[jk]).max() <= 1e-12 * np.abs(wj[jk]).max()


@pytest.fixture
def ctxs():
    hs = [frg.frg_create(0, b) for b in BUDGETS.values()]
    yield hs
    torch.cuda.synchronize()
    for h in hs:
        frg.frg_destroy(h)


@pytest.mark.parametrize("reg", [EXP, LIT])
@pytest.mark.parametrize("n_r", [1, 40, 130])
def test_points_in_no_panel(ctxs, n_r, reg):
    print(f"[case] lpa in no panel, {n_r} nodes, reg {reg}", flush=True)
    n = 129  # differences of slope * rho are exact: both masses at 2^e
    rho = np.arange(n) * (0.5 / (n - 1))
    for e in (-40, -27, 33, 34, 50):
        slope = (2.0 ** e - 1.0) * rho
        for few in (3, n // 2, n):  # that many points there, the others at 1 + 1.5
            U = np.where(np.arange(n) < few, slope,
                         slope[min(few, n - 1)] + 1.5 * (rho - rho[min(few, n - 1)]))
            check(ctxs, reg, n_r, 4, U)
        check(ctxs, reg, n_r, 1, slope)
    check(ctxs, reg, n_r, 2, 3.0 * 2.0 ** 33 * rho ** 2)  # across 2^34
    check(ctxs, reg, n_r, 2, (rho + 0.1) ** 2, t=-14.0)


@pytest.mark.parametrize("n", [4, 65, 20000])  # 20000: a wave's worth of points each
def test_sizes(ctxs, n):
    print(f"[case] lpa with and without the table, {n} points", flush=True)
    check(ctxs, EXP, 64, 4, 1.5 * (np.linspace(0.0, 0.5, n) - 0.02) ** 2)


def test_wide_radial_rule(ctxs):
    """Nodes beyond 2^18 k^2: no expansion above the panels."""
    rho = np.linspace(0.0, 0.5, 200)
    for t in (0.0, -14.0):
        check(ctxs, EXP, 64, 4, (rho + 0.1) ** 2, t=t, q_max=1000.0)


def test_time_in_no_panel():
    """1024 points and nodes: a lane with all nodes of its point took 15 times as long
    as a point in the panels."""
    us = {}
    n = 1024
    U, D, J = dev((np.linspace(0.0, 0.5, n) + 0.1) ** 2), dev(np.zeros(n)), dev(np.zeros(7 * n))
    lpa = frg.make_lpa(n_radial=1024, n_grid=n, N=4)
    for budget in BUDGETS:
        ctx = frg.frg_create(0, BUDGETS[budget])
        try:
            for t in (-0.5, -13.0):
                best = float("inf")
                for _ in range(4):
                    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                    a.record()
                    for _ in range(100):
                        frg.frg_flow_rhs(ctx, lpa, t, U, D, J)
                    b.record()
                    torch.cuda.synchronize()
                    best = min(best, a.elapsed_time(b) * 10.0)
                us[budget, t] = best
        finally:
            torch.cuda.synchronize()
            frg.frg_destroy(ctx)
    print(f"  us per call {us}")
    assert max(us.values()) < 4 * us["table", -0.5]
