"""Segmented tables: term sorts with half a wave per part of the radial nodes (up
to 32 angular nodes) and with a whole one, and runs of every length modulo the
16 lanes that take them, against the cache-streamed form."""
import numpy as np
import pytest

from paper_2607_24908_amd import frg, workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_r,n_a", [(1, 1), (3, 32), (7, 5), (8, 32), (9, 31), (13, 17), (65, 32),
                                     (130, 3), (5, 33)])
@pytest.mark.parametrize("n_rows,n_p", [(1, 1), (5, 67)])
def test_parts_and_runs(n_r, n_a, n_rows, n_p):
    print(f"[case] segmented parts {n_r}x{n_a}, {n_rows} rows, {n_p} momenta", flush=True)
    ctx = frg.frg_create(0)
    try:
        rng = np.random.Generator(np.random.PCG64(n_r * 100 + n_a + n_p))
        s_max = 676.0
        q = frg.make_quad(3, frg.FRG_REG_EXP, 1.0, 6.0, n_r, n_a)
        dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
        g = dev(workloads.tab_rows(n_rows, 20483, s_max))
        p = dev(np.concatenate([[0.0], 10 ** rng.uniform(-3, np.log10(20.0), n_p - 1)]))
        out = []
        frg.frg_tune_set(ctx, "tab_lds_nodes", 2)
        for seg in (1, 0):
            frg.frg_tune_set(ctx, "tab_seg", seg)
            o = torch.full((n_p, n_rows), float("nan"), dtype=torch.float64, device="cuda")
            frg.frg_integrate_tab(ctx, q, g, s_max, p, o)
            torch.cuda.synchronize()
            out.append(o.cpu().numpy())
        # the same terms summed in another order: n u relative, all of one sign
        assert np.all(np.abs(out[0] - out[1]) <= 1e-13 * np.abs(out[1]))
        assert np.all(out[0] != 0.0)
    finally:
        torch.cuda.synchronize()
        frg.frg_destroy(ctx)
