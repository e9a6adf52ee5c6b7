"""Status and state of the adjoint solve on both forms of its step.

Grids of up to 512 partial sums of 256 cells take two kernels per step, larger
ones four.  A breakdown (a state that is an energy maximum along its field:
negative curvature) must come out as MM_ENONFINITE on either side, and leave
the context able to solve the next problem with the result of a fresh one bit
for bit; an exhausted budget reports exactly that many iterations, at odd and
even counts, and a poll interval that ends early or late changes nothing.
"""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

GRIDS = [(5, 3, 1), (512, 256, 1), (512, 257, 1)]


def context(n, H, **options):
    from paper_1405_2728_amd import Context
    ctx = Context("fp64")
    for k, v in options.items():
        ctx.set_option(k, v)
    ctx.set_geometry(0, *n, 5e-9, 5e-9, 5e-9)
    ctx.set_material(0, 8e5, 1.3e-11, 500.0)
    ctx.set_field(0, (H, 0.0, 0.0))
    return ctx


def vectors(n):
    m = torch.zeros((3,) + n[::-1], dtype=torch.float64, device="cuda")
    m[0] = 1.0
    g = torch.Generator("cuda").manual_seed(3)
    rhs = torch.randn(m.shape, dtype=torch.float64, device="cuda", generator=g)
    rhs[0] = 0.0                       # tangent to m = x
    return m, rhs


@pytest.mark.parametrize("n", GRIDS)
def test_breakdown_is_reported_and_leaves_no_trace(n):
    from paper_1405_2728_amd import MMError
    m, rhs = vectors(n)
    with context(n, 2e6) as ctx:
        fresh = ctx.adjoint_solve(0, m, rhs, tol=1e-8, max_iter=200)
    with context(n, -2e6) as ctx:      # energy maximum: negative curvature
        with pytest.raises(MMError) as e:
            ctx.adjoint_solve(0, m, rhs, tol=1e-8, max_iter=50)
        assert e.value.code == -4
        bad = rhs.clone()
        bad[1, 0, 0, 0] = float("nan")
        with pytest.raises(MMError) as e:
            ctx.adjoint_solve(0, m, bad, tol=1e-8, max_iter=50)
        assert e.value.code == -4
        ctx.set_field(0, (2e6, 0.0, 0.0))
        again = ctx.adjoint_solve(0, m, rhs, tol=1e-8, max_iter=200)
    assert torch.equal(again[0], fresh[0]) and again[1:] == fresh[1:]


@pytest.mark.parametrize("n", GRIDS)
def test_budget_and_poll_interval(n):
    m, rhs = vectors(n)
    zero = torch.zeros_like(rhs)
    with context(n, 2e6) as ctx:
        full = ctx.adjoint_solve(0, m, rhs, tol=1e-8, max_iter=200)
        assert full[3] == 0 and full[1] > 5
        for k in (0, 1, 2, 5):
            lam, iters, res, status = ctx.adjoint_solve(0, m, rhs, tol=1e-14, max_iter=k)
            assert status == 1 and iters == k and res > 1e-14
        lam, iters, res, status = ctx.adjoint_solve(0, m, zero, tol=1e-8, max_iter=50)
        assert status == 0 and iters == 0 and float(lam.abs().max()) == 0.0
    for poll in (1, 3, 7):
        with context(n, 2e6, poll_every=poll) as ctx:
            other = ctx.adjoint_solve(0, m, rhs, tol=1e-8, max_iter=200)
        assert torch.equal(other[0], full[0]) and other[1:] == full[1:]
