"""Finite-volume flux from polynomial panels, on the GPU against the oracle: cell
counts at the edges of the fused solve's waves (63 cells each, eight waves per
pass), masses that sweep the panels (2^-14 <= (m^2 + k^2)/k^2 < 2^22) and leave
them on both sides."""
import numpy as np
import pytest

import oracle
from paper_2607_24908_amd import frg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

D, N_R, SMAX = 3, 48, 2.0
LOW = -16  # smallest exponent of (m^2 + k^2)/k^2


def states(n):
    """Cell values of four flows at k = 1: u/sigma + 1 from 2^LOW to 1, from 1 to
    2^24, near 1, and a jump of 2^25 in the middle."""
    sigma = (np.arange(n) + 0.5) * SMAX / n
    w = sigma / SMAX
    u = np.stack([sigma * (2.0 ** (LOW * (1 - w)) - 1.0), sigma * (2.0 ** (24 * w) - 1.0),
                  sigma * (0.1 + 0.3 * np.sin(5 * sigma)), sigma.copy()])
    u[3, n // 2:] += 2.0 ** 25
    return u


@pytest.mark.parametrize("N", [1, 4])
@pytest.mark.parametrize("n", [2, 3, 62, 63, 64, 126, 127, 505, 1100])
def test_panels_and_wave_edges(n, N):
    print(f"[case] fvlpa panels n={n} N={N}", flush=True)
    ctx = frg.frg_create(0)
    try:
        reg = frg.FRG_REG_EXP
        u = states(n)
        fv = frg.make_fvlpa(D, N, reg, N_R, 1.0, 6.0, n, SMAX)
        U = torch.tensor(u, dtype=torch.float64, device="cuda")
        out = torch.full_like(U, float("nan"))
        dt = torch.full((len(u),), float("nan"), dtype=torch.float64, device="cuda")
        frg.frg_fvlpa_rhs(ctx, fv, 0.0, U, out, dt)
        torch.cuda.synchronize()
        want, wdt, dead = oracle.fvlpa_rhs(D, N, reg, N_R, 1.0, 6.0, SMAX, 0.0, u,
                                           allow_domain=True)
        got, gdt = out.cpu().numpy(), dt.cpu().numpy()
        assert np.array_equal(np.isnan(got).all(axis=1), dead != 0)
        ok = dead == 0
        # a difference quotient of fluxes of the size of N F_1 at the smallest mass,
        # whose m^2 + k^2 >= 2^LOW carries the rounding of m^2 ~ 1
        rtol = 1e-12 + 8 * 2.0 ** (-53 - LOW)
        F1 = oracle.threshold(D, reg, 1.0, 6.0, N_R, 1, [2.0 ** LOW - 1.0])[0]
        sc = np.maximum(N * F1 * n / SMAX, np.abs(want[ok]))
        err = (np.abs(got[ok] - want[ok]) / sc).max()
        edt = np.abs(gdt[ok] / wdt[ok] - 1.0).max()
        print(f"  alive {ok.sum()}/4, max scaled err {err:.3e}, step estimate {edt:.3e}")
        assert err < rtol and edt < rtol
        outs = []
        for fused in (1, 0):
            frg.frg_tune_set(ctx, "fv_persistent", fused)
            V = U.clone()
            tr = torch.empty(len(u), dtype=torch.float64, device="cuda")
            frg.frg_fvlpa_solve(ctx, fv, -3 * 0.25 * wdt[ok].min(), 3, V, tr)
            torch.cuda.synchronize()
            outs.append((V.cpu().numpy(), tr.cpu().numpy()))
        assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
        assert np.isfinite(outs[0][0]).all()
    finally:
        torch.cuda.synchronize()
        frg.frg_destroy(ctx)


def test_budget_that_cannot_spare_the_panels():
    """A context of 1 MiB keeps to the sums of the radial nodes: within rounding of
    one with panels, right-hand sides and solves (fused and by launches the same
    bits), and a flow whose footprint the budget just holds is still served."""
    print("[case] fvlpa and lpa without panels", flush=True)
    n, N = 127, 4
    u = states(n)[1:3]
    fv = frg.make_fvlpa(D, N, frg.FRG_REG_EXP, N_R, 1.0, 6.0, n, SMAX)
    lpa = frg.make_lpa(d=3, N=2, n_grid=200)
    U0 = 1.5 * (np.arange(200) * (0.5 / 199) - 0.02) ** 2
    res = []
    for budget in (0, 1 << 20):
        ctx = frg.frg_create(0, budget)
        try:
            U = torch.tensor(u, dtype=torch.float64, device="cuda")
            out, dt = torch.empty_like(U), torch.empty(2, dtype=torch.float64, device="cuda")
            frg.frg_fvlpa_rhs(ctx, fv, 0.0, U, out, dt)
            sol = []
            for fused in (1, 0):
                frg.frg_tune_set(ctx, "fv_persistent", fused)
                V, tr = U.clone(), torch.empty(2, dtype=torch.float64, device="cuda")
                frg.frg_fvlpa_solve(ctx, fv, -1e-6, 5, V, tr)
                sol.append(V)
            L = torch.tensor(U0, dtype=torch.float64, device="cuda")
            dL, J = torch.empty_like(L), torch.empty(7 * 200, dtype=torch.float64, device="cuda")
            frg.frg_flow_rhs(ctx, lpa, -0.1, L, dL, J)
            torch.cuda.synchronize()
            assert torch.equal(sol[0], sol[1])
            res.append([x.cpu().numpy() for x in (out, dt, sol[0], dL, J)])
        finally:
            torch.cuda.synchronize()
            frg.frg_destroy(ctx)
    for a, b in zip(*res):  # the second flow is outside its domain: NaN rates
        ok = np.isfinite(a)
        assert ok.any() and np.array_equal(ok, np.isfinite(b))
        assert np.abs(a - b)[ok].max() <= 1e-12 * np.abs(a[ok]).max()
    big = frg.make_lpa(d=3, N=2, n_grid=1024)
    table = 4096  # the radial table of 64 nodes
    ctx = frg.frg_create(0, frg.frg_flow_footprint(big) + table)
    try:
        small = frg.make_lpa(d=3, N=2, n_grid=64)
        L = torch.zeros(64, dtype=torch.float64, device="cuda")
        frg.frg_flow_rhs(ctx, small, 0.0, L, torch.empty_like(L))
        torch.cuda.synchronize()
        out = np.zeros(1024)
        t = frg.frg_submit(ctx, frg.make_request(big, 6.0, 0.05, -0.05, 1e-6, 1e-9, out))
        while frg.frg_poll(ctx, t)[0] == frg.FRG_PENDING:
            pass
        assert np.isfinite(out).all() and (out != 0.0).any()
    finally:
        frg.frg_destroy(ctx)
