"""Small thin films that one workgroup holds (double precision).

Grids at the edges of the held shapes (rows of 1, 32, 33 and 64 cells,
columns of 1, 16, 17 and 32, one and two layers) and just beyond them:
effective field, energy and field terms against the oracle (1e-10, the
library's parity bound), runs and sweeps against the oracle's iterates
(1e-8, the bound of the other kernels' iterate tests), and the consistency
of single steps, continued runs and graph replay with one run.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from oracle import fields as ofields, minimizer as omin

pytestmark = pytest.mark.gpu

GRIDS = [(1, 1, 1), (2, 1, 2), (32, 1, 1), (1, 32, 1), (7, 3, 1), (32, 16, 1), (33, 16, 1),
         (64, 16, 1), (65, 16, 1), (32, 17, 1), (32, 32, 1), (31, 33, 1), (32, 16, 2),
         (33, 15, 2), (12, 7, 2), (9, 5, 3), (64, 17, 1), (50, 13, 1)]
D = (5e-9, 4e-9, 6e-9)
H = np.array([3e4, -2e3, 1e3])


def setup(ctx, n, ku=500.0, sample=0):
    ctx.set_geometry(sample, *n, *D)
    if isinstance(ku, np.ndarray):
        ctx.set_material(sample, 8e5, 1.3e-11, 0.0, (1, 0.2, 0), ku_map=torch.tensor(ku, device="cuda"))
    else:
        ctx.set_material(sample, 8e5, 1.3e-11, ku, (1, 0.2, 0))
    ctx.set_field(sample, H)


@pytest.mark.parametrize("n", GRIDS)
def test_field_energy_and_terms(n):
    from paper_1405_2728_amd import Context
    rng = np.random.default_rng(2)
    m0 = synth.random_unit(*n, rng)
    ku = 500.0 * (1.0 + 0.1 * rng.standard_normal(n[::-1]))
    P = ofields.Problem(*n, *D, Ms=8e5, A=1.3e-11, Ku=ku, u=(1, 0.2, 0), H_ext=H)
    t = P.field_terms(m0)
    ref = P.heff(m0)
    with Context("fp64") as ctx:
        setup(ctx, n, ku)
        m = torch.tensor(m0, device="cuda")
        out = ctx.heff(0, m)
        static = ctx.heff_static(0, m, torch.empty_like(m))
        terms = ctx.field_terms(0, m)
        E, parts = ctx.energy(0, m)
        scale = np.max(np.abs(ref))
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-10 * scale
        assert torch.equal(out, static)
        for a, k in zip(terms, ("demag", "exchange", "anisotropy")):
            assert np.max(np.abs(a.cpu().numpy() - t[k])) <= 1e-10 * max(scale, np.max(np.abs(t[k])))
        ref_parts = P.energy_terms(m0)
        size = sum(abs(v) for v in ref_parts)
        assert abs(E - sum(ref_parts)) <= 1e-10 * size
        for a, b in zip(parts, ref_parts):
            assert abs(a - b) <= 1e-10 * size
        assert np.array_equal(m.cpu().numpy(), m0)


@pytest.mark.parametrize("n", [(20, 10, 1), (33, 16, 1), (32, 30, 1), (12, 7, 2)])
def test_run_matches_the_oracle_and_its_parts(n):
    from paper_1405_2728_amd import Context
    m0 = synth.uniform_with_noise((1, 0.3, 0), *n, 1e-3, np.random.default_rng(4))
    P = ofields.Problem(*n, *D, Ms=8e5, A=1.3e-11, Ku=500.0, u=(1, 0.2, 0), H_ext=H)
    ref = omin.minimize(P, m0, tol=0.0, max_iter=10)
    with Context("fp64") as ctx:
        setup(ctx, n)
        m = torch.tensor(m0, device="cuda")
        r = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=10)
        assert r["iters"] == 10 and r["heff_evals"] == 11
        assert np.max(np.abs(m.cpu().numpy() - ref["m"])) < 1e-8
        # single steps, a continued run and graph replay: the same iterates
        ms = torch.tensor(m0, device="cuda")
        ctx.reset(0)
        for _ in range(10):
            ctx.minimize_step(0, ms)
        assert torch.equal(ms, m)
        full = torch.tensor(m0, device="cuda")
        rf = ctx.minimize_to_tol(0, full, tol=1e-7, max_iter=5000)
        assert rf["converged"]
        part = torch.tensor(m0, device="cuda")
        ctx.minimize_to_tol(0, part, tol=0.0, max_iter=37)
        rc = ctx.minimize_continue(0, part, tol=1e-7, max_iter=5000)
        assert torch.equal(part, full) and rc["iters"] == rf["iters"]
    stream = torch.cuda.Stream()
    with Context("fp64", stream=stream) as ctx, torch.cuda.stream(stream):
        ctx.set_option("use_graph", 1)
        setup(ctx, n)
        g = torch.tensor(m0, device="cuda")
        ctx.minimize_to_tol(0, g, tol=1e-7, max_iter=5000)
        stream.synchronize()
        assert torch.equal(g, full)
    assert omin.minimize(P, full.cpu().numpy(), tol=1.001e-7, max_iter=1)["iters"] == 0


def test_sweep_with_a_small_sample_and_errors():
    from paper_1405_2728_amd import Context, MMError
    grids = [(32, 16, 1), (64, 32, 1), (20, 10, 2)]
    rng = np.random.default_rng(8)
    m0 = [synth.uniform_with_noise((1, 0.1, 0), *n, 1e-3, rng) for n in grids]
    fields = np.array([[k * 5e3, 4e2, 0.0] for k in (3, 2, 1)])
    with Context("fp64", n_samples=3) as ctx:
        for k, n in enumerate(grids):
            setup(ctx, n, sample=k)
        ms = [torch.tensor(m, device="cuda") for m in m0]
        avg, iters, rc = ctx.hysteresis_sweep(ms, np.stack([fields] * 3), tol=1e-6, max_iter=20000)
        assert rc == 0
    for k, n in enumerate(grids):
        with Context("fp64") as ctx:
            setup(ctx, n)
            m = torch.tensor(m0[k], device="cuda")
            a1, i1, _ = ctx.hysteresis_sweep([m], fields, tol=1e-6, max_iter=20000)
            assert np.array_equal(a1[0], avg[k]) and np.array_equal(i1[0], iters[k])
            assert torch.equal(m, ms[k])
    with Context("fp64") as ctx:
        setup(ctx, grids[0])
        bad = torch.tensor(m0[0], device="cuda")
        bad[0, 0, 3, 5] = float("nan")
        with pytest.raises(MMError) as e:
            ctx.minimize_to_tol(0, bad, tol=1e-6, max_iter=100)
        assert e.value.code == -4
        ok = torch.tensor(m0[0], device="cuda")
        assert ctx.minimize_to_tol(0, ok, tol=1e-6, max_iter=20000)["converged"]
