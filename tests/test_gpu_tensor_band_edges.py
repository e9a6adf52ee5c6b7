"""Demag tensor of the device set-up where offsets lie exactly on a band edge.

With cubic cells whole-number triples put offsets exactly 6, 16 and 40 cells
away, off the axes as well: (24, 32, 0) and (0, 24, 32) are 40 h away.  The
field of films and a small bulk grid that hold such offsets is compared with
the oracle's (bound 1e-10 of its maximum, the library's parity bound); an
offset written by neither kernel would leave memory's former contents in the
tensor.  Flat and elongated cells, whose closed-form band covers many cells or
the whole grid, with odd and even numbers of offsets in the band's box.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from oracle import fields as ofields

pytestmark = pytest.mark.gpu

CUBIC = (5e-9, 5e-9, 5e-9)
GRIDS = [((45, 45, 1), CUBIC), ((25, 33, 2), CUBIC), ((33, 25, 3), (3e-9, 3e-9, 3e-9)),
         ((1, 1, 1), CUBIC), ((3, 1, 1), CUBIC), ((70, 21, 1), (1e-9, 1e-9, 1e-8)),
         ((71, 23, 1), (1e-9, 1e-9, 5e-9)), ((9, 9, 7), (1e-9, 2e-9, 2e-8)),
         ((2, 25, 33), CUBIC), ((26, 17, 33), (1e-8 / 3, 1e-8 / 3, 1e-8 / 3))]


@pytest.mark.parametrize("n,d", GRIDS)
def test_field_against_the_oracle(n, d):
    from paper_1405_2728_amd import Context
    m0 = synth.random_unit(*n, np.random.default_rng(17))
    ref = ofields.Problem(*n, *d, Ms=8e5, A=1.3e-11, Ku=500.0).h_demag(m0)
    with Context("fp64") as ctx:
        ctx.set_geometry(0, *n, *d)
        ctx.set_material(0, 8e5, 1.3e-11, 500.0)
        hd, _, _ = ctx.field_terms(0, torch.tensor(m0, device="cuda"))
    assert np.max(np.abs(hd.cpu().numpy() - ref)) <= 1e-10 * np.max(np.abs(ref))
