"""Grids and vertex diagrams with many masses: values at the nodes of the mass
panels, interpolated.

A panel is a factor of 16 in x = sig (m^2 + k^2); its interpolant through 32
nodes is the discrete sum to 2e-18 relative, so the results meet the bar of the
direct form (1e-12 against the oracle) and agree with it to rounding (1e-13, as
the other forms do).  Masses at and next to the panel ends and on a node, in
two to twelve panels, outside every panel and outside the domain; momenta
outside the coefficient form; one to several batches' worth of workgroups per
momentum; captured streams (which take the direct form)."""
import numpy as np
import pytest

import oracle
from paper_2607_24908_amd import frg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EXP, LIT = frg.FRG_REG_EXP, frg.FRG_REG_LITIM
RTOL, XTOL = 1e-12, 1e-13


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available()
    h = frg.frg_create(0)
    yield h
    torch.cuda.synchronize()
    frg.frg_destroy(h)


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def grid(ctx, quad, p, m2, form=0):
    out = torch.full((len(p), len(m2)), -7.0, dtype=torch.float64, device="cuda")
    frg.frg_tune_set(ctx, "grid_form", form)
    try:
        frg.frg_integrate_grid(ctx, quad, dev(p), dev(m2), out)
        torch.cuda.synchronize()
    finally:
        frg.frg_tune_set(ctx, "grid_form", 0)
    return out.cpu().numpy()


def vertex(ctx, quad, n_phi, p1, p2, c12, m2, form=0):
    out = torch.full((len(p1), len(m2)), -7.0, dtype=torch.float64, device="cuda")
    frg.frg_tune_set(ctx, "grid_form", form)
    try:
        frg.frg_integrate_vertex(ctx, quad, n_phi, dev(p1), dev(p2), dev(c12), dev(m2), out)
        torch.cuda.synchronize()
    finally:
        frg.frg_tune_set(ctx, "grid_form", 0)
    return out.cpu().numpy()


def masses(kind, n, k):
    """n masses, unsorted; delta = m^2 + k^2 in units where sig k^2 is in [1, 2)."""
    rng = np.random.Generator(np.random.PCG64(n))
    k2 = k * k
    sig = 2.0 ** (1 - np.frexp(k2)[1])
    if kind == "two":          # two panels, their ends and their neighbours
        ends = np.array([1.0, np.nextafter(1.0, 0.0), 1 / 16, 16.0 * (1 - 2.0 ** -52), 0.25, 4.0])
        x = np.concatenate([ends, 16.0 ** rng.uniform(-1.0, 1.0, n - ends.size)])
    elif kind == "twelve":     # every panel, and both sides of the outermost ends
        ends = np.array([2.0 ** -24, 2.0 ** -25, 2.0 ** 24, 2.0 ** 24 * (1 - 2.0 ** -53)])
        x = np.concatenate([ends, 2.0 ** rng.uniform(-24.0, 24.0, n - ends.size)])
    elif kind == "one":        # one point many times, with a few neighbours
        x = np.full(n, 1.7)
        x[::7] = 1.0 + 14.9 * rng.random(x[::7].size)
    else:                      # "mixed": masses outside the domain and beyond the panels
        x = 16.0 ** rng.uniform(-1.0, 1.0, n)
        x[3], x[n // 2], x[n - 1] = -1.0, 1e-12, 1e9
        x[5] = 0.0
    m2 = rng.permutation(x) / sig - k2
    return m2


GRIDS = [  # d, reg, n_r, n_a, n_p, n_m, kind
    (3, EXP, 128, 32, 700, 128, "two"), (4, LIT, 100, 24, 517, 131, "mixed"),
    (3, EXP, 64, 48, 200, 800, "twelve"), (4, EXP, 33, 5, 1100, 513, "one"),
    (5, LIT, 17, 70, 300, 400, "two"), (3, EXP, 1, 9, 5000, 200, "two"),
    (3, EXP, 300, 44, 97, 257, "mixed"), (3, LIT, 64, 16, 400, 768, "twelve"),
]


@pytest.mark.parametrize("d,reg,n_r,n_a,n_p,n_m,kind", GRIDS)
def test_grid_matches_direct_form_and_oracle(ctx, d, reg, n_r, n_a, n_p, n_m, kind):
    print(f"[case] mass nodes grid d={d} reg={reg} {n_r}x{n_a} {n_p}x{n_m} {kind}", flush=True)
    k = 0.8
    rng = np.random.Generator(np.random.PCG64(n_p))
    p = 10.0 ** rng.uniform(-4.0, 1.3, n_p)
    p[:3] = 0.0, 1e-9, 3e8        # 3e8: beyond the range of the 16-term groups
    m2 = masses(kind, n_m, k)
    quad = frg.make_quad(d, reg, k, 6 * k, n_r, n_a)
    got, direct = grid(ctx, quad, p, m2), grid(ctx, quad, p, m2, form=3)
    bad = ~(m2 + k * k > 0.0)
    assert np.array_equal(np.isnan(got), np.broadcast_to(bad, got.shape))
    good = ~bad
    sel = np.concatenate([[0, 1, 2], np.arange(3, n_p, max(1, n_p // 9))])
    want = oracle.integrate_grid(d, reg, k, 6 * k, n_r, n_a, p[sel], m2[good], threads=8)
    err = np.abs(got[sel][:, good] - want.reshape(sel.size, -1)) / want.reshape(sel.size, -1)
    print(f"  against the oracle {err.max():.2e}, against the direct form "
          f"{np.max(np.abs(got[:, good] / direct[:, good] - 1)):.2e}")
    assert err.max() < RTOL
    assert np.all(np.abs(got[:, good] - direct[:, good]) <= XTOL * direct[:, good])


VERTICES = [(3, EXP, 48, 8, 16, 256, 256, "two"), (4, LIT, 24, 6, 8, 400, 300, "mixed"),
            (3, EXP, 20, 3, 33, 300, 384, "two"), (5, EXP, 48, 8, 16, 9, 130, "one"),
            (3, LIT, 48, 8, 16, 60, 800, "twelve")]


@pytest.mark.parametrize("d,reg,n_r,n_a,n_phi,n_c,n_m,kind", VERTICES)
def test_vertex_matches_direct_form_and_oracle(ctx, d, reg, n_r, n_a, n_phi, n_c, n_m, kind):
    print(f"[case] mass nodes vertex d={d} reg={reg} {n_r}x{n_a}x{n_phi} {n_c}x{n_m} {kind}",
          flush=True)
    k = 0.9
    rng = np.random.Generator(np.random.PCG64(n_c))
    p1, p2 = 10.0 ** rng.uniform(-3, 1, n_c), 10.0 ** rng.uniform(-3, 1, n_c)
    c12 = rng.uniform(-1.0, 1.0, n_c)
    p1[0], p2[1], c12[2] = 0.0, 0.0, 1.0
    p1[4], c12[5] = -0.5, 1.5      # outside the domain
    m2 = masses(kind, n_m, k)
    quad = frg.make_quad(d, reg, k, 6 * k, n_r, n_a)
    got, direct = (vertex(ctx, quad, n_phi, p1, p2, c12, m2, f) for f in (0, 1))
    bad = ~(m2 + k * k > 0.0)
    nan = np.broadcast_to(bad, got.shape).copy()
    nan[4:6] = True
    assert np.array_equal(np.isnan(got), nan)
    assert np.all(np.abs(got - direct)[~nan] <= XTOL * np.abs(direct[~nan]))
    ia = np.array([0, 1, 2, 3, n_c - 1])
    ib = np.flatnonzero(~bad)[::max(1, n_m // 40)]
    P1, P2, C = (np.repeat(v[ia], ib.size) for v in (p1, p2, c12))
    want = oracle.integrate_vertex(d, reg, k, 6 * k, n_r, n_a, n_phi, P1, P2, C,
                                   np.tile(m2[ib], ia.size), threads=8)
    err = np.abs(got[np.ix_(ia, ib)].ravel() - want) / np.abs(want)
    print(f"  against the oracle {err.max():.2e}")
    assert err.max() < RTOL


def test_results_do_not_depend_on_the_batch(ctx):
    """One, two and four workgroups per momentum (many, some and few momenta)
    give a momentum the same bits; a mass alone in its panel and the record of a
    mass outside the domain survive the interpolated form."""
    k = 1.0
    quad = frg.make_quad(3, EXP, k, 6 * k, 128, 32)
    rng = np.random.Generator(np.random.PCG64(1))
    p = 10.0 ** rng.uniform(-4.0, 1.3, 1030)
    m2 = masses("two", 512, k)
    full = grid(ctx, quad, p, m2)
    assert np.array_equal(grid(ctx, quad, p[:400], m2), full[:400])
    assert np.array_equal(grid(ctx, quad, p[100:250], m2), full[100:250])
    frg.frg_stream_status(ctx, allow_domain=True)  # clears what earlier calls recorded
    m2[7] = -2.0
    grid(ctx, quad, p[:300], m2)
    assert frg.frg_stream_status(ctx, allow_domain=True) == frg.FRG_E_DOMAIN


def test_captured_and_two_stream_calls(ctx):
    """A captured call replays with the values of an eager one (to rounding:
    the capture takes the direct form); calls on two streams share the
    context's buffers without mixing."""
    k = 1.0
    quad = frg.make_quad(3, EXP, k, 6 * k, 64, 16)
    rng = np.random.Generator(np.random.PCG64(2))
    p = dev(10.0 ** rng.uniform(-4.0, 1.3, 2000))
    ms = [dev(masses("two", 400, k)), dev(masses("two", 401, k))]
    outs = [torch.zeros(2000, m.numel(), dtype=torch.float64, device="cuda") for m in ms]
    streams = [torch.cuda.Stream() for _ in ms]
    ref = []
    for m, o in zip(ms, outs):
        frg.frg_integrate_grid(ctx, quad, p, m, o)
        torch.cuda.synchronize()
        ref.append(o.clone())
    for _ in range(5):
        for o in outs:
            o.zero_()
        torch.cuda.synchronize()
        for m, o, s in zip(ms, outs, streams):
            frg.frg_integrate_grid(ctx, quad, p, m, o, stream=s)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, ref))
    frg.frg_integrate_grid(ctx, quad, p, ms[0], outs[0], stream=streams[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=streams[0]):
        frg.frg_integrate_grid(ctx, quad, p, ms[0], outs[0], stream=streams[0])
    for _ in range(3):
        outs[0].zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.all((outs[0] - ref[0]).abs() <= XTOL * ref[0])
