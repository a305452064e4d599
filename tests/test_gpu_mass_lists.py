"""Mass lists of interpolated grids and vertex diagrams that take more than the eight
tiles of a workgroup's registers: masses of -0.9..10 k^2 in three panels (k = 0.9), lists
over five to twelve panels, interpolated or not, long lists beyond the panels, with
one to four workgroups per momentum.  Against the oracle and the direct form, the same
bits for any number of momenta, and not slower than the direct form."""
import numpy as np
import pytest

import oracle
from paper_2607_24908_amd import frg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EXP, LIT = frg.FRG_REG_EXP, frg.FRG_REG_LITIM
RTOL, XTOL = 1e-12, 1e-13  # of the other mass-node tests


@pytest.fixture(scope="module")
def ctx():
    h = frg.frg_create(0)
    yield h
    torch.cuda.synchronize()
    frg.frg_destroy(h)


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def masses(kind, n, k):
    """Unsorted masses: -0.9..10 k^2, or (m^2 + k^2)/k^2 from 2^lo to 2^hi with some
    outside the domain."""
    rng = np.random.Generator(np.random.PCG64(n))
    if kind == "near":
        return rng.permutation(np.linspace(-0.9, 10.0, n)) * k * k
    lo, hi = kind
    x = 2.0 ** rng.permutation(np.linspace(lo, hi, n))
    x[n // 3], x[n - 1] = -0.5, 0.0
    return (x - 1.0) * k * k


def call(ctx, kind, form, *a):
    out = torch.full((a[-2].numel(), a[-1].numel()) if kind == "grid" else
                     (a[2].numel(), a[-1].numel()), -7.0, dtype=torch.float64, device="cuda")
    frg.frg_tune_set(ctx, "grid_form", form)
    try:
        (frg.frg_integrate_grid if kind == "grid" else frg.frg_integrate_vertex)(ctx, *a, out)
        torch.cuda.synchronize()
    finally:
        frg.frg_tune_set(ctx, "grid_form", 0)
    return out.cpu().numpy()


LISTS = [("near", 131), ("near", 190), ((-2, 15), 160), ((-20, 20), 200), ((-20, 20), 300),
         ((-20, 20), 384), ((-20, 20), 512), ((-24, 24), 450), ((10, 44), 1500)]


@pytest.mark.parametrize("reg,n_r,n_a", [(EXP, 128, 32), (LIT, 100, 24)])
@pytest.mark.parametrize("kind,n_m", LISTS)
def test_grid_lists(ctx, kind, n_m, reg, n_r, n_a):
    print(f"[case] mass lists grid {kind} {n_m} reg={reg}", flush=True)
    k, n_p = 0.9, 1040
    rng = np.random.Generator(np.random.PCG64(n_m))
    p = 10.0 ** rng.uniform(-4.0, 1.3, n_p)
    p[0], p[1], p[2] = 0.0, -1.0, 3e8  # at zero, outside the domain, beyond the form
    m2 = masses(kind, n_m, k)
    quad = frg.make_quad(3, reg, k, 6 * k, n_r, n_a)
    P, M = dev(p), dev(m2)
    got, direct = call(ctx, "grid", 0, quad, P, M), call(ctx, "grid", 3, quad, P, M)
    bad = ~(m2 + k * k > 0.0)
    nan = np.broadcast_to(bad, got.shape).copy()
    nan[1] = True
    assert np.array_equal(np.isnan(got), nan)
    assert np.all(np.abs(got - direct)[~nan] <= XTOL * np.abs(direct[~nan]))
    ia, ib = np.array([0, 2, 3, 500, 1039]), np.flatnonzero(~bad)[::max(1, n_m // 40)]
    want = oracle.integrate_grid(3, reg, k, 6 * k, n_r, n_a, p[ia], m2[ib], threads=8)
    assert (np.abs(got[np.ix_(ia, ib)] / want.reshape(ia.size, -1) - 1.0)).max() < RTOL
    # two and four workgroups per momentum (one above, 1040 momenta), of the calls that
    # are large enough for this form: 2.5e8 momenta x masses x nodes in lane slots
    nodes = 128 * n_a  # 100 radial nodes take two rows of 64 lanes
    for part in (slice(0, 510), slice(100, 356)):
        n = part.stop - part.start
        if n * n_m * nodes >= 2.5e8:
            assert np.array_equal(call(ctx, "grid", 0, quad, P[part], M), got[part],
                                  equal_nan=True)


@pytest.mark.parametrize("n_phi", [16, 5])
@pytest.mark.parametrize("kind,n_m", LISTS)
def test_vertex_lists(ctx, kind, n_m, n_phi):
    print(f"[case] mass lists vertex {kind} {n_m} n_phi={n_phi}", flush=True)
    k, n_c = 0.9, 1100
    rng = np.random.Generator(np.random.PCG64(n_m + 1))
    p1, p2 = 10.0 ** rng.uniform(-3, 1, n_c), 10.0 ** rng.uniform(-3, 1, n_c)
    c12 = rng.uniform(-1.0, 1.0, n_c)
    p1[0], c12[1] = 0.0, 1.5  # c12[1]: outside the domain
    m2 = masses(kind, n_m, k)
    quad = frg.make_quad(3, EXP, k, 6 * k, 40, 8)
    a = [dev(v) for v in (p1, p2, c12)]
    M = dev(m2)
    got, direct = (call(ctx, "vertex", f, quad, n_phi, *a, M) for f in (0, 1))
    bad = ~(m2 + k * k > 0.0)
    nan = np.broadcast_to(bad, got.shape).copy()
    nan[1] = True
    assert np.array_equal(np.isnan(got), nan)
    assert np.all(np.abs(got - direct)[~nan] <= XTOL * np.abs(direct[~nan]))
    ia, ib = np.array([0, 2, 700]), np.flatnonzero(~bad)[::max(1, n_m // 30)]
    P1, P2, C = (np.repeat(v[ia], ib.size) for v in (p1, p2, c12))
    want = oracle.integrate_vertex(3, EXP, k, 6 * k, 40, 8, n_phi, P1, P2, C,
                                   np.tile(m2[ib], ia.size), threads=8)
    assert np.abs(got[np.ix_(ia, ib)].ravel() / want - 1.0).max() < RTOL


@pytest.mark.parametrize("kind,n_m", [("near", 190), ((-20, 20), 512)])
def test_not_slower_than_the_direct_form(ctx, kind, n_m):
    """1024 momenta, 128 x 32 nodes: 1.07 and 1.3 times as long as the direct form where
    every eight tiles took a pass over the table of their own."""
    k = 0.9
    rng = np.random.Generator(np.random.PCG64(3))
    p, m2 = dev(10.0 ** rng.uniform(-4.0, 1.3, 1024)), dev(masses(kind, n_m, k))
    quad = frg.make_quad(3, EXP, k, 6 * k, 128, 32)
    out = torch.zeros(1024, n_m, dtype=torch.float64, device="cuda")
    us = {}
    for form in (0, 3):
        frg.frg_tune_set(ctx, "grid_form", form)
        best = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(20):
                frg.frg_integrate_grid(ctx, quad, p, m2, out)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50.0)
        us[form] = best
    frg.frg_tune_set(ctx, "grid_form", 0)
    print(f"  {kind} {n_m}: {us[0]:.1f} us, direct form {us[3]:.1f} us")
    assert us[0] < us[3]
