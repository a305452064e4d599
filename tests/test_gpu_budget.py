"""The buffers of interpolated grids against the context's HBM budget: they are given back
to a call that needs their room, a call's form does not hang on what other calls
hold, and without room the direct form answers."""
import numpy as np
import pytest

from paper_2607_24908_amd import frg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BUDGET = 512 << 20
N_P, N_M, N_R, N_A = 200, 128, 256, 48  # 6 MB of buffers, a share is 8


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def grid(ctx, form=0):
    rng = np.random.Generator(np.random.PCG64(1))
    p, m2 = dev(10.0 ** rng.uniform(-4.0, 1.3, N_P)), dev(rng.uniform(-0.9, 10.0, N_M))
    out = torch.zeros(N_P, N_M, dtype=torch.float64, device="cuda")
    frg.frg_tune_set(ctx, "grid_form", form)
    frg.frg_integrate_grid(ctx, frg.make_quad(3, 0, 1.0, 6.0, N_R, N_A), p, m2, out)
    torch.cuda.synchronize()
    frg.frg_tune_set(ctx, "grid_form", 0)
    return out


def staged(ctx, left):
    """A host-memory call whose staging takes the budget but for `left` bytes."""
    n_m = 100
    n_p = (BUDGET - left) // (17 * n_m + 8)
    out = np.zeros((n_p, n_m))
    frg.frg_integrate_grid(ctx, frg.make_quad(3, 0, 1.0, 6.0, 4, 2), np.linspace(0.1, 2.0, n_p),
                           np.linspace(0.0, 3.0, n_m), out, mem=frg.FRG_MEM_HOST)
    assert np.all(out > 0.0)


@pytest.fixture
def ctx():
    h = frg.frg_create(0, BUDGET)
    yield h
    torch.cuda.synchronize()
    frg.frg_destroy(h)


def test_buffers_are_given_back(ctx):
    direct = grid(ctx, form=3)
    first = grid(ctx)
    assert not torch.equal(first, direct)  # interpolated
    staged(ctx, 800_000)  # fits beside the tables alone
    assert torch.equal(grid(ctx, form=3), direct)
    again = grid(ctx)  # no room left: the direct form
    assert torch.all((again - first).abs() <= 1e-13 * first)


def test_form_does_not_hang_on_other_buffers(ctx):
    other = frg.frg_create(0, BUDGET)
    try:
        staged(other, 32 << 20)
        assert torch.equal(grid(ctx), grid(other))
    finally:
        torch.cuda.synchronize()
        frg.frg_destroy(other)


def test_small_shares_take_fewer_momenta_at_a_time():
    """The same bits in one batch of momenta and in several."""
    rng = np.random.Generator(np.random.PCG64(2))
    p, m2 = dev(10.0 ** rng.uniform(-4.0, 1.3, 6000)), dev(rng.uniform(-0.9, 10.0, 512))
    quad = frg.make_quad(3, 0, 1.0, 6.0, 64, 16)
    outs = []
    for budget in (0, 2 << 30):  # 32 MB: two batches and more
        ctx = frg.frg_create(0, budget)
        try:
            out = torch.zeros(6000, 512, dtype=torch.float64, device="cuda")
            frg.frg_integrate_grid(ctx, quad, p, m2, out)
            torch.cuda.synchronize()
            outs.append(out)
        finally:
            frg.frg_destroy(ctx)
    assert torch.equal(*outs)
