"""Full 3-D demag path at the edges of its padded z and y lengths.

The z pass packs 8, 4, 2 or 1 pencils into a wave by the padded length (64,
128, 256, 512) and precision; layer counts that just fit and just miss each
length are compared with the oracle's field (1e-10 of its maximum in double
precision, 1e-5 in the mixed form: the library's parity bounds), alone and
in a batched sweep of 3-D samples, which must equal the per-sample sweep bit
for bit.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from oracle import fields as ofields

pytestmark = pytest.mark.gpu

GRIDS = [(6, 5, 5), (3, 33, 31), (5, 4, 32), (4, 3, 33), (3, 65, 7), (6, 2, 64), (2, 3, 65),
         (3, 2, 128), (2, 5, 129), (1, 2, 256)]


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("mixed", 1e-5)])
def test_field_at_length_edges(n, prec, tol):
    from paper_1405_2728_amd import Context
    d = (5e-9, 4e-9, 3e-9)
    m0 = synth.random_unit(*n, np.random.default_rng(11))
    H = np.array([2e4, -1e3, 5e3])
    P = ofields.Problem(*n, *d, Ms=8e5, A=1.3e-11, Ku=500.0, H_ext=H)
    ref = P.heff(m0)
    with Context(prec) as ctx:
        ctx.set_geometry(0, *n, *d)
        ctx.set_material(0, 8e5, 1.3e-11, 500.0)
        ctx.set_field(0, H)
        out = ctx.heff(0, torch.tensor(m0, device="cuda")).cpu().numpy()
    assert np.max(np.abs(out - ref)) <= tol * np.max(np.abs(ref))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_batched_3d_samples_equal_single_ones(prec):
    from paper_1405_2728_amd import Context
    grids = [(70, 5, 6), (66, 9, 33), (40, 33, 65)]
    rng = np.random.default_rng(5)
    m0 = [synth.uniform_with_noise((1, 0.2, 0), *n, 1e-2, rng) for n in grids]
    H = np.array([[[3e4, 1e3, 0.0], [2.5e4, 1e3, 0.0]]] * len(grids))
    res = []
    for batched in (1, 0):
        with Context(prec, n_samples=len(grids)) as ctx:
            ctx.set_option("batched", batched)
            for k, n in enumerate(grids):
                ctx.set_geometry(k, *n, 5e-9, 5e-9, 5e-9)
                ctx.set_material(k, 8e5, 1.3e-11, 500.0)
            ms = [torch.tensor(m, device="cuda") for m in m0]
            ctx.hysteresis_sweep(ms, H, tol=1e-9, max_iter=20)
            res.append([m.cpu().numpy() for m in ms])
    for a, b in zip(*res):
        assert np.array_equal(a, b)
