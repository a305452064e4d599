"""LPA right-hand sides from polynomial panels: grids at the edges of the 64-point
workgroups, masses over the range of the panels (2^-26 <= (m^2 + k^2)/k^2 < 2^34)
and beyond them on both sides, batches at the edge of what a launch takes as
arguments."""
import numpy as np
import pytest

import oracle
from paper_2607_24908_amd import frg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [4, 5, 6, 33, 63, 64, 65, 66, 127, 128, 129, 257, 1025]


def state(n, i):
    """U on n points of [0, 0.5] at k = 1; on 2^m + 1 points the differences of the
    first are exact."""
    rho = np.arange(n) * (0.5 / (n - 1))
    if i % 3 == 0 and (n - 1) & (n - 2) == 0:
        return (2.0 ** -16 - 1.0) * rho  # both masses give x = 2^-16
    if i % 3 == 1:
        return 2.0 ** 24 * rho ** 2  # x from 1 to 3 2^24
    return 1.5 * (rho - 0.02) ** 2


def dev(a):
    return torch.tensor(a, dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("n_flows", [1, 13, 24, 25, 39])
def test_batches_and_panel_edges(n_flows):
    ctx = frg.frg_create(0)
    try:
        lpas, Us, Ds, Js = [], [], [], []
        for i in range(n_flows):
            n = SIZES[i % len(SIZES)]
            lpas.append(frg.make_lpa(d=3, N=(1, 2, 4)[i % 3], reg=frg.FRG_REG_EXP, n_radial=40,
                                     n_grid=n))
            Us.append(dev(state(n, i)))
            Ds.append(dev(np.full(n, np.nan)))
            Js.append(dev(np.full(7 * n, np.nan)))
        print(f"[case] lpa panels, {n_flows} flows", flush=True)
        frg.frg_flow_rhs_batch(ctx, lpas, [0.0] * n_flows, Us, Ds, Js)
        torch.cuda.synchronize()
        worst = 0.0
        for l, U, D, J in zip(lpas, Us, Ds, Js):
            d1, j1 = torch.zeros_like(D), torch.zeros_like(J)
            frg.frg_flow_rhs(ctx, l, 0.0, U, d1, j1)
            torch.cuda.synchronize()
            assert torch.equal(d1, D) and torch.equal(j1, J)
            want, wj, rc = oracle.lpa_rhs(3, l.N, frg.FRG_REG_EXP, 40, 6.0, 1.0, 0.5,
                                          U.cpu().numpy())
            assert rc == 0
            err = np.abs(D.cpu().numpy() / want - 1.0).max()
            wj = np.asarray(wj).ravel()
            ej = np.abs(J.cpu().numpy() - wj).max() / np.abs(wj).max()
            worst = max(worst, err, ej)
            assert err < 1e-12 and ej < 1e-12
        print(f"  max rel err {worst:.2e}")
    finally:
        torch.cuda.synchronize()
        frg.frg_destroy(ctx)


@pytest.mark.parametrize("reg", [frg.FRG_REG_EXP, frg.FRG_REG_LITIM])
@pytest.mark.parametrize("e", [-32, -27, -26, -25, 32, 33, 34, 40])
def test_edges_of_the_panels(e, reg):
    """Both masses of every point at (m^2 + k^2)/k^2 = 2^e (exact differences), N = 1
    and 4, with the other points of the second flow inside the panels."""
    print(f"[case] lpa panels 2^{e}", flush=True)
    ctx = frg.frg_create(0)
    try:
        n = 129
        rho = np.arange(n) * (0.5 / (n - 1))
        slope = (2.0 ** e - 1.0) * rho
        mixed = np.where(np.arange(n) < n // 2, slope, slope[n // 2] + 1.5 * (rho - rho[n // 2]))
        for U, N in ((slope, 1), (slope, 4), (mixed, 4)):
            want, wj, rc = oracle.lpa_rhs(3, N, reg, 40, 6.0, 1.0, 0.5, U, allow_domain=True)
            dU, J = torch.empty(n, dtype=torch.float64, device="cuda"), dev(np.empty(7 * n))
            frg.frg_flow_rhs(ctx, frg.make_lpa(d=3, N=N, reg=reg, n_radial=40, n_grid=n), 0.0,
                             dev(U), dU, J)
            frg.frg_stream_status(ctx, allow_domain=True)
            got, wj = dU.cpu().numpy(), np.asarray(wj).ravel()
            ok = np.isfinite(want)  # the kink may leave the domain
            assert np.array_equal(ok, np.isfinite(got)) and ok.any()
            assert np.abs(got[ok] / want[ok] - 1.0).max() < 1e-12
            jk = np.isfinite(wj)
            assert np.abs(J.cpu().numpy()[jk] - wj[jk]).max() <= 1e-12 * np.abs(wj[jk]).max()
    finally:
        torch.cuda.synchronize()
        frg.frg_destroy(ctx)


def test_destroy_while_the_first_batch_is_prepared():
    """Flows whose calls a batch has taken when the context goes (the first batch
    builds the tables of 1024 radial nodes, longer than a call polls) outlive that
    batch; a later context works."""
    print("[case] destroy during the first batch", flush=True)
    for i in range(3):
        c = frg.frg_create(0)
        outs = [np.zeros(256) for _ in range(8)]
        lpa = frg.make_lpa(d=3, N=2, n_radial=1024, q_max_over_k=6.0 + 0.1 * i, n_grid=256)
        for o in outs:
            frg.frg_submit(c, frg.make_request(lpa, 6.0, 0.05, -9.0, 1e-8, 1e-10, o))
        frg.frg_destroy(c)
        assert all(np.all(np.isfinite(o)) for o in outs)
    c = frg.frg_create(0)
    try:
        U = torch.zeros(64, dtype=torch.float64, device="cuda")
        D = torch.full_like(U, float("nan"))
        frg.frg_flow_rhs(c, frg.make_lpa(d=3, N=1, n_grid=64), 0.0, U, D)
        torch.cuda.synchronize()
        assert torch.isfinite(D).all()
    finally:
        frg.frg_destroy(c)
