"""Bulk grids with more than 512 cells along x (double precision).

Their rows take the long wave transforms (1280, 1536, 1792 or 2048 padded
points) around the packed y and z passes of the full 3-D path.  Grids at the
edges of each length, also thin ones sent to the 3-D path, are compared with
the oracle's field (1e-10 of its maximum, the library's parity bound), its
first iterates (1e-8, the bound of the other iterate tests) and the field
with powers of two only (1e-12 of its maximum where the lengths differ: both
are the exact convolution up to rounding).
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from oracle import fields as ofields, minimizer as omin

pytestmark = pytest.mark.gpu

D = (5e-9, 4e-9, 3e-9)
H = np.array([2e4, -1e3, 5e3])
GRIDS = [((513, 2, 5), 0), ((520, 3, 5), 0), ((640, 2, 6), 0), ((641, 3, 5), 0), ((700, 2, 6), 0),
         ((768, 2, 5), 0), ((769, 2, 5), 0), ((896, 3, 5), 0), ((897, 2, 5), 0), ((1024, 2, 5), 0),
         ((600, 3, 2), 2), ((900, 2, 1), 2)]


def context(n, path, **options):
    from paper_1405_2728_amd import Context
    ctx = Context("fp64")
    ctx.set_option("demag_path", path)
    for k, v in options.items():
        ctx.set_option(k, v)
    ctx.set_geometry(0, *n, *D)
    ctx.set_material(0, 8e5, 1.3e-11, 500.0)
    ctx.set_field(0, H)
    return ctx


@pytest.mark.parametrize("n,path", GRIDS)
def test_field_and_iterates(n, path):
    m0 = synth.uniform_with_noise((1, 0.2, 0), *n, 0.1, np.random.default_rng(5))
    P = ofields.Problem(*n, *D, Ms=8e5, A=1.3e-11, Ku=500.0, H_ext=H)
    ref = P.heff(m0)
    scale = np.max(np.abs(ref))
    it = omin.minimize(P, m0, tol=0.0, max_iter=6)
    with context(n, path) as ctx:
        m = torch.tensor(m0, device="cuda")
        h = ctx.heff(0, m)
        assert np.max(np.abs(h.cpu().numpy() - ref)) <= 1e-10 * scale
        r = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=6)
        assert r["iters"] == 6
        assert np.max(np.abs(m.cpu().numpy() - it["m"])) < 1e-8
        assert abs(r["energy"] / it["energy"] - 1) < 1e-8
    if n[0] <= 896:
        with context(n, path, mixed_radix=0) as ctx:
            h2 = ctx.heff(0, torch.tensor(m0, device="cuda"))
        assert float((h2 - h).abs().max()) <= 1e-12 * scale


@pytest.mark.parametrize("n", [(520, 3, 5), (800, 4, 6), (1000, 3, 5)])
def test_runs_agree_bit_for_bit(n):
    """Fused finish, finish kernel, graph replay and a continued run."""
    m0 = synth.uniform_with_noise((1, 0.3, 0), *n, 0.1, np.random.default_rng(9))
    out = []
    for opts in ({}, {"fused_finish": 0}):
        with context(n, 0, poll_every=8, **opts) as ctx:
            m = torch.tensor(m0, device="cuda")
            r = ctx.minimize_to_tol(0, m, tol=0.0, max_iter=30)
            out.append((r, m))
    with context(n, 0, poll_every=8) as ctx:
        m = torch.tensor(m0, device="cuda")
        ctx.minimize_to_tol(0, m, tol=0.0, max_iter=13)
        out.append((ctx.minimize_continue(0, m, tol=0.0, max_iter=30), m))
    for r, m in out[1:]:
        assert torch.equal(m, out[0][1])
        assert r["torque"] == out[0][0]["torque"] and r["energy"] == out[0][0]["energy"]
