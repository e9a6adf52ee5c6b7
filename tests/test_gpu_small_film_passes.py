"""Small films on the separate passes.

A forced rows_per_block asks for the x passes of that tile, so films that one
workgroup would hold (double precision, up to 1024 cells) then take the
separate passes, with their LDS transforms at the film's generic lengths.
They are compared with the one-workgroup kernel (fields to 1e-12 of their
maximum: both are the exact convolution up to rounding; ten updates to 1e-8,
the bound of the other iterate tests) and among their tiles, alone and in a
sweep beside batched samples, which must equal the sweep of the samples one by
one bit for bit.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth

pytestmark = pytest.mark.gpu

D = (5e-9, 4e-9, 6e-9)


def run(n, m0, **options):
    from paper_1405_2728_amd import Context
    with Context("fp64") as ctx:
        for k, v in options.items():
            ctx.set_option(k, v)
        ctx.set_geometry(0, *n, *D)
        ctx.set_material(0, 8e5, 1.3e-11, 500.0, (1, 0.2, 0))
        ctx.set_field(0, (3e4, -2e3, 1e3))
        if options.get("rows_per_block"):
            assert ctx.rows_per_block(0) == options["rows_per_block"]
        m = torch.tensor(m0, device="cuda")
        h = ctx.heff(0, m)
        e, _ = ctx.energy(0, m)
        ctx.minimize_to_tol(0, m, tol=0.0, max_iter=10)
        ctx.profile("all")
        ctx.heff(0, m)
        launches = {k: v[1] for k, v in ctx.profile_read().items() if v[1]}
        return h, e, m, launches


@pytest.mark.parametrize("n", [(1, 1, 1), (7, 3, 1), (20, 10, 1), (33, 16, 1), (32, 30, 1),
                               (12, 7, 2)])
def test_tiles_take_the_separate_passes(n):
    m0 = synth.uniform_with_noise((1, 0.3, 0), *n, 1e-2, np.random.default_rng(4))
    h, e, m, one = run(n, m0)
    assert one == {"xf": 1}
    scale = float(h.abs().max())
    for R in [r for r in (1, 2, 4) if r <= n[1]]:   # tiles of the wave and the LDS passes
        hr, er, mr, passes = run(n, m0, rows_per_block=R)
        assert passes == {"xf": 1, "yz_thin": 1, "xil": 1}
        assert float((hr - h).abs().max()) <= 1e-12 * scale
        assert abs(er - e) <= 1e-12 * abs(e) + 1e-30
        assert float((mr - m).abs().max()) < 1e-8
    hv, _, _, passes = run(n, m0, yz_variant=0)
    assert passes == {"xf": 1, "yz_thin": 1, "xil": 1}
    assert float((hv - h).abs().max()) <= 1e-12 * scale


def test_separate_passes_run_without_timing():
    n = (20, 10, 1)
    m0 = synth.random_unit(*n, np.random.default_rng(6))
    assert not torch.equal(run(n, m0)[0], run(n, m0, rows_per_block=2)[0])


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_sweep_beside_batched_samples(prec):
    from paper_1405_2728_amd import Context
    grids = [(64, 32, 1), (20, 10, 1), (70, 33, 1), (12, 7, 2)]
    rng = np.random.default_rng(12)
    m0 = [synth.uniform_with_noise((1, 0.1, 0), *n, 1e-3, rng) for n in grids]
    fields = np.array([[k * 5e3, 4e2, 0.0] for k in (3, 2, 1)])
    res = []
    for batched in (0, 1):
        with Context(prec, n_samples=len(grids)) as ctx:
            ctx.set_option("batched", batched)
            for k, n in enumerate(grids):
                ctx.set_option("rows_per_block", 2 if n[0] * n[1] < 1000 else 0)
                ctx.set_geometry(k, *n, 5e-9, 5e-9, 5e-9)
                ctx.set_material(k, 8e5, 1.3e-11, 500.0)
            ms = [torch.tensor(m, device="cuda") for m in m0]
            avg, iters, rc = ctx.hysteresis_sweep(ms, np.stack([fields] * len(grids)), tol=1e-6,
                                                  max_iter=20000)
            assert rc == 0
            res.append((avg, iters, ms))
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])
    assert all(torch.equal(a, b) for a, b in zip(res[0][2], res[1][2]))
