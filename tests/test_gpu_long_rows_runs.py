"""Runs of double-precision films beyond 512 padded points along x or y.

Every padded row length of the long wave transforms (1280, 1536, 1792, 2048
points: half lengths 640 to 1024) and every column length (640, 768, 896, 1024)
with one to three layers: first iterates against the oracle's (1e-8, the bound
of the other iterate tests), line-search runs with rejected trials against the
oracle's, and bit for bit the same run with the finish fused into the forward
pass or as a kernel, from a replayed graph, and continued from a checkpoint.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from oracle import fields as ofields, minimizer as omin

pytestmark = pytest.mark.gpu

D = (5e-9, 4e-9, 6e-9)
H = np.array([3e4, -2e3, 1e3])
ROWS = [(520, 3, 1), (700, 2, 2), (800, 5, 3), (1000, 3, 1), (1024, 2, 4)]
COLUMNS = [(2 if nz > 1 else 5, ny, nz) for ny in (300, 384, 440, 500) for nz in (1, 2, 3)]
BOTH = [(520, 300, 1), (700, 385, 2)]


def context(n, stream=None, **options):
    from paper_1405_2728_amd import Context
    ctx = Context("fp64", stream=stream)
    for k, v in options.items():
        ctx.set_option(k, v)
    ctx.set_geometry(0, *n, *D)
    ctx.set_material(0, 8e5, 1.3e-11, 500.0, (1, 0.2, 0))
    ctx.set_field(0, H)
    return ctx


def problem(n):
    return ofields.Problem(*n, *D, Ms=8e5, A=1.3e-11, Ku=500.0, u=(1, 0.2, 0), H_ext=H)


@pytest.mark.parametrize("n", ROWS + COLUMNS + BOTH)
def test_iterates(n):
    m0 = synth.uniform_with_noise((1, 0.3, 0.1), *n, 0.1, np.random.default_rng(21))
    ref = omin.minimize(problem(n), m0, tol=0.0, max_iter=6)
    with context(n) as ctx:
        m = torch.tensor(m0, device="cuda")
        r = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=6)
    assert r["iters"] == 6
    assert np.max(np.abs(m.cpu().numpy() - ref["m"])) < 1e-8
    assert abs(r["energy"] / ref["energy"] - 1) < 1e-8
    assert abs(r["torque"] / ref["torque"] - 1) < 1e-8


@pytest.mark.parametrize("n", ROWS)
def test_line_search_iterates(n):
    # a first step far too long: trials are rejected and shortened
    m0 = synth.uniform_with_noise((1, 0.3, 0.1), *n, 0.2, np.random.default_rng(17))
    tau0 = 3.0 / 8e5
    ref = omin.minimize_ls(problem(n), m0, tol=0.0, max_iter=10, tau0=tau0)
    assert ref["backtracks"] >= 1
    with context(n, line_search=1, tau0=tau0) as ctx:
        m = torch.tensor(m0, device="cuda")
        r = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=10)
    assert r["iters"] == 10 and r["heff_evals"] == ref["heff_evals"]
    assert np.max(np.abs(m.cpu().numpy() - ref["m"])) < 1e-8
    assert abs(r["energy"] / ref["energy"] - 1) < 1e-8


@pytest.mark.parametrize("n", ROWS + COLUMNS[1:2] + BOTH)
def test_the_same_run_bit_for_bit(n):
    m0 = synth.uniform_with_noise((1, 0.3, 0.1), *n, 0.1, np.random.default_rng(23))
    opts = {"poll_every": 8}
    K = 45
    with context(n, **opts) as ctx:
        ref = torch.tensor(m0, device="cuda")
        r = ctx.minimize_to_tol(0, ref, tol=0.0, max_iter=K)
    with context(n, fused_finish=0, **opts) as ctx:
        m = torch.tensor(m0, device="cuda")
        rf = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=K)
        assert torch.equal(m, ref) and rf == r
    stream = torch.cuda.Stream()
    with context(n, stream=stream, use_graph=1, **opts) as ctx, torch.cuda.stream(stream):
        m = torch.empty_like(ref)
        for _ in range(2):                     # the second run replays the kept graph
            m.copy_(torch.tensor(m0, device="cuda"))
            rg = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=K)
            stream.synchronize()
            assert torch.equal(m, ref) and rg == r
    with context(n, **opts) as ctx:
        m = torch.tensor(m0, device="cuda")
        ctx.minimize_to_tol(0, m, tol=0.0, max_iter=13)
        blob = ctx.state_save(0)
    with context(n, **opts) as ctx:
        ctx.state_load(0, blob)
        rc = ctx.minimize_continue(0, m, tol=0.0, max_iter=K)
        assert torch.equal(m, ref) and rc == r


@pytest.mark.parametrize("n", [(520, 30, 1), (1000, 20, 2)])
def test_a_bounded_wait_that_gives_up_is_reported(n):
    """Blocks told to give up at once (fin_spin 0) end the run with MM_ESTATE;
    the context runs as before afterwards."""
    from paper_1405_2728_amd import MMError
    m0 = synth.uniform_with_noise((1, 0.3, 0.1), *n, 0.1, np.random.default_rng(23))
    with context(n) as ctx:
        ref = torch.tensor(m0, device="cuda")
        ctx.minimize_to_tol(0, ref, tol=0.0, max_iter=20)
        ctx.set_option("fin_spin", 0)
        m = torch.tensor(m0, device="cuda")
        with pytest.raises(MMError) as e:
            ctx.minimize_to_tol(0, m, tol=0.0, max_iter=20)
        assert e.value.code == -5
        ctx.set_option("fin_spin", 1 << 22)
        m = torch.tensor(m0, device="cuda")
        ctx.minimize_to_tol(0, m, tol=0.0, max_iter=20)
        assert torch.equal(m, ref)
