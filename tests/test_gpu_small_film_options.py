"""Options that must not change what a small film computes.

Double-precision films of up to 1024 cells run in one workgroup.  Timing the
kernels and turning the line search on (which concerns runs only) leave their
fields, energies and, for timing, runs the same bit for bit; the timer records
the launches such a run makes, under "xf".  Line-search runs, which take the
separate passes at the film's own padded lengths, follow the oracle's iterates
(1e-8, the bound of the other iterate tests).
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from oracle import fields as ofields, minimizer as omin

pytestmark = pytest.mark.gpu

GRIDS = [(20, 10, 1), (33, 16, 1), (32, 30, 1), (12, 7, 2)]
D = (5e-9, 4e-9, 6e-9)
H = np.array([3e4, -2e3, 1e3])


def context(n, **options):
    from paper_1405_2728_amd import Context
    ctx = Context("fp64")
    for k, v in options.items():
        ctx.set_option(k, v)
    ctx.set_geometry(0, *n, *D)
    ctx.set_material(0, 8e5, 1.3e-11, 500.0, (1, 0.2, 0))
    ctx.set_field(0, H)
    return ctx


def start(n):
    return synth.uniform_with_noise((1, 0.3, 0), *n, 1e-2, np.random.default_rng(4))


@pytest.mark.parametrize("n", GRIDS)
def test_timing_leaves_the_run_and_times_its_launches(n):
    m0 = start(n)
    out = []
    for timed in (False, True):
        with context(n) as ctx:
            if timed:
                ctx.profile("all")
            m = torch.tensor(m0, device="cuda")
            h = ctx.heff(0, m)
            e = ctx.energy(0, m)
            r = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=70)
            part = torch.tensor(m0, device="cuda")
            ctx.minimize_to_tol(0, part, tol=0.0, max_iter=37)
            if timed:
                ctx.profile(None)           # timing ends within the run
            ctx.minimize_continue(0, part, tol=0.0, max_iter=70)
            assert torch.equal(part, m)
            out.append((h, e, r, m))
            if timed:
                prof = ctx.profile_read()
                # field, energy, 71 evaluations in batches of 32, 38 in two
                assert prof["xf"][1] == 2 + 3 + 2 and prof["xf"][0] > 0.0
                assert sum(v[1] for k, v in prof.items() if k != "xf") == 0
                b = ctx.kernel_bytes(0)
                assert b["xf"] > 0 and b["yz_thin"] == b["xil"] == b["finish"] == 0
    (h0, e0, r0, m1), (h1, e1, r1, m2) = out
    assert torch.equal(h0, h1) and e0 == e1 and r0 == r1 and torch.equal(m1, m2)


@pytest.mark.parametrize("n", GRIDS)
def test_line_search_option(n):
    # a first step far too long: trials are rejected and shortened
    m0 = synth.uniform_with_noise((1, 0.3, 0.1), *n, 0.2, np.random.default_rng(17))
    tau0 = 3.0 / 8e5
    m = torch.tensor(m0, device="cuda")
    with context(n) as ctx:
        h, e = ctx.heff(0, m), ctx.energy(0, m)
    P = ofields.Problem(*n, *D, Ms=8e5, A=1.3e-11, Ku=500.0, u=(1, 0.2, 0), H_ext=H)
    ref = omin.minimize_ls(P, m0, tol=0.0, max_iter=10, tau0=tau0)
    assert ref["backtracks"] >= 1
    with context(n, line_search=1, tau0=tau0) as ctx:
        assert torch.equal(ctx.heff(0, m), h) and ctx.energy(0, m) == e
        r = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=10)
        assert r["iters"] == 10 and r["heff_evals"] == ref["heff_evals"]
        assert np.max(np.abs(m.cpu().numpy() - ref["m"])) < 1e-8


@pytest.mark.parametrize("n", GRIDS)
def test_checkpoint_continues_bit_for_bit(n):
    m0 = start(n)
    with context(n) as ctx:
        full = torch.tensor(m0, device="cuda")
        r = ctx.minimize_to_tol(0, full, tol=0.0, max_iter=70)
    with context(n) as ctx:
        m = torch.tensor(m0, device="cuda")
        ctx.minimize_to_tol(0, m, tol=0.0, max_iter=29)
        blob = ctx.state_save(0)
    with context(n) as ctx:
        ctx.state_load(0, blob)
        c = ctx.minimize_continue(0, m, tol=0.0, max_iter=70)
        assert torch.equal(m, full) and c == r
