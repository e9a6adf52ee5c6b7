"""Demag tensor of the device set-up at the edges of its distance bands.

The set-up evaluates offsets below 40 h (h the largest cell edge) with one
wave per offset inside a box that holds them, and those beyond with 8 lanes
per offset; the closed form ends at 6 h and the 6-point rule at 16 h.  Grids
whose extent ends just below, at and beyond these edges along each axis, with
cubic and flat cells, are compared through the effective field with the
oracle's tensor (bound 1e-10 of the field's maximum, the library's parity
bound: it covers the closed form's cancellation in double precision).
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth
from oracle import fields as ofields

pytestmark = pytest.mark.gpu

GRIDS = [
    ((6, 1, 1), (5e-9, 5e-9, 5e-9)), ((7, 2, 1), (5e-9, 5e-9, 5e-9)),
    ((17, 3, 2), (5e-9, 5e-9, 5e-9)), ((40, 1, 1), (5e-9, 5e-9, 5e-9)),
    ((41, 1, 1), (5e-9, 5e-9, 5e-9)), ((42, 2, 1), (5e-9, 5e-9, 5e-9)),
    ((44, 3, 2), (5e-9, 5e-9, 5e-9)), ((1, 44, 1), (5e-9, 5e-9, 5e-9)),
    ((2, 3, 45), (5e-9, 5e-9, 5e-9)), ((30, 30, 1), (5e-9, 5e-9, 5e-9)),
    ((100, 9, 1), (5e-9, 5e-9, 2e-9)), ((90, 5, 2), (2e-9, 5e-9, 3e-9)),
    ((9, 70, 1), (5e-9, 3e-9, 1e-9)),
]


@pytest.mark.parametrize("n,d", GRIDS)
def test_field_across_the_bands(n, d):
    from paper_1405_2728_amd import Context
    m0 = synth.random_unit(*n, np.random.default_rng(7))
    P = ofields.Problem(*n, *d, Ms=8e5, A=1.3e-11, Ku=500.0)
    ref = P.h_demag(m0)
    with Context("fp64") as ctx:
        ctx.set_geometry(0, *n, *d)
        ctx.set_material(0, 8e5, 1.3e-11, 500.0)
        hd, _, _ = ctx.field_terms(0, torch.tensor(m0, device="cuda"))
        hd = hd.cpu().numpy()
    assert np.max(np.abs(hd - ref)) <= 1e-10 * np.max(np.abs(ref))
