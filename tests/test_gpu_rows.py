"""Several rows per workgroup: results collected in groups of 64, 32 or 16 lanes (one,
two or four rows) with more momenta per wave than a group has lanes, and flows in
groups of four whose last one is ragged, with fewer waves than a full workgroup."""
import numpy as np
import pytest

from paper_2607_24908_amd import frg, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("n_p", [1, 15, 16, 17, 33, 64, 65, 2100])
def test_more_momenta_per_wave_than_lanes_of_a_row(n_p):
    print(f"[case] rows, {n_p} momenta", flush=True)
    ctx = frg.frg_create(0)
    try:
        rng = np.random.Generator(np.random.PCG64(n_p))
        n_rows, s_max = 1030 if n_p < 2000 else 70, 400.0  # enough rows for 64 momenta per wave
        q = frg.make_quad(3, frg.FRG_REG_EXP, 1.0, 6.0, 24, 8)
        g = dev(workloads.tab_rows(n_rows, 130, s_max))
        p = 10 ** rng.uniform(-3, 1.2, n_p)
        p[n_p // 2] = -1.0  # outside the domain: NaN for every row
        outs = []
        for rb, W in ((1, 4), (2, 16), (4, 16), (2, 1), (4, 2), (0, 16)):
            frg.frg_tune_set(ctx, "tab_rb", rb)
            frg.frg_tune_set(ctx, "tab_rW", W)
            frg.frg_tune_set(ctx, "tab_pw", 64)
            o = torch.full((n_p, n_rows), 7.0, dtype=torch.float64, device="cuda")
            frg.frg_integrate_tab(ctx, q, g, s_max, dev(p), o)
            frg.frg_stream_status(ctx, allow_domain=True)
            outs.append(o.cpu().numpy())
        assert np.isnan(outs[0][n_p // 2]).all()
        assert np.isfinite(np.delete(outs[0], n_p // 2, axis=0)).all()
        assert not (outs[0] == 7.0).any()
        for o in outs[1:]:
            assert np.array_equal(o, outs[0], equal_nan=True)
    finally:
        torch.cuda.synchronize()
        frg.frg_destroy(ctx)


@pytest.mark.parametrize("n_flows,n_s", [(1, 33), (2, 40), (3, 257), (66, 256), (67, 256), (129, 130),
                                         (5, 2300), (2, 3100), (9, 4097)])
def test_flow_groups(n_flows, n_s):
    """Flows of a batch and alone, fused and by two launches: the same bits."""
    print(f"[case] flow groups {n_flows} x {n_s}", flush=True)
    ctx = frg.frg_create(0)
    try:
        rng = np.random.Generator(np.random.PCG64(n_flows + n_s))
        pf = frg.make_pflow(3, frg.FRG_REG_EXP, 24, 8, 1.0, 6.0, n_s, 40.0)
        lam3, lam4 = rng.uniform(0.2, 2.5, n_flows), rng.uniform(0.0, 6.0, n_flows)
        S0 = np.repeat(rng.uniform(0.2, 1.0, n_flows)[:, None], n_s, axis=1)
        S0[-1] -= 2.5  # the last flow of the ragged group is outside the domain

        def solve(sel, fused):
            frg.frg_tune_set(ctx, "pflow_fused", fused)
            S = dev(S0[sel])
            tr = torch.zeros(len(S0[sel]), dtype=torch.float64, device="cuda")
            frg.frg_pflow_solve(ctx, pf, dev(lam3[sel]), dev(lam4[sel]), -0.15, 3, S, tr)
            torch.cuda.synchronize()
            return S.cpu().numpy(), tr.cpu().numpy()

        S, tr = solve(slice(None), 1)
        S2, tr2 = solve(slice(None), 0)
        assert np.array_equal(S, S2) and np.array_equal(tr, tr2)
        assert tr[-1] == 0.0 and np.array_equal(S[-1], S0[-1])
        if n_flows > 1:
            assert (tr[:-1] == -0.15).all() and np.isfinite(S).all()
        for i in {0, n_flows // 2, n_flows - 1}:
            Si, ti = solve(slice(i, i + 1), 1)
            assert np.array_equal(Si[0], S[i]) and ti[0] == tr[i]
    finally:
        torch.cuda.synchronize()
        frg.frg_destroy(ctx)
