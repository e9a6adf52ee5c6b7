"""Scratch use of the kernels that double-precision contexts launch beyond
those of test_lib_kernels.py (no GPU needed).

The packed 3-D passes, the long wave transforms, the one-workgroup films, the
x passes of several rows per block, the split tensor set-up and the two-kernel
conjugate-gradient step must use no scratch memory and spill no vector
register, each in every instance that a dispatch can reach.
"""

from test_lib_kernels import kernels  # noqa: F401  (fixture)

WAVE = range(1, 9)
LONG = (10, 12, 14, 16)
REACHED = (
    ["k_xf_w<double, %d, %s>" % (v, f) for v in WAVE for f in ("true", "false")]
    + ["k_xf_wr<double, %d, %s>" % (v, f) for v in WAVE for f in ("true", "false")]
    + ["k_xil_w<double, %d>" % v for v in WAVE] + ["k_xil_wr<double, %d>" % v for v in WAVE]
    + ["k_xf_long<%d, %s>" % (v, f) for v in LONG for f in ("true", "false")]
    + ["k_xil_long<%d>" % v for v in LONG]
    + ["k_yz_long<%d, %d>" % (v, nz) for v in LONG for nz in (1, 2, 3)]
    + ["k_%s_pk<%d>" % (k, v) for k in ("y3_fwd", "z3", "y3_inv") for v in (1, 2, 4, 8)]
    + ["k_w3_p<double, %d, true>" % s for s in (-1, 0, 1)]
    + ["k_x_wp<double, %s, %d>" % (inv, rc) for inv in ("true", "false") for rc in (0, 1)]
    + ["k_small<1, 32, 32>", "k_small<1, 64, 32>", "k_small<1, 32, 64>", "k_small<2, 32, 32>"]
    + ["k_newell_near", "k_newell_far", "k_cg_update_own", "k_cg_direction_own",
       "k_finish_stage1", "k_finish_stage1_b", "k_finish_b"]
)


def test_reached_instances_use_no_scratch(kernels):  # noqa: F811
    missing = [k for k in REACHED if k not in kernels]
    assert not missing, missing
    used = {k: kernels[k] for k in REACHED
            if kernels[k].get("vgpr_spill_count", 0) or kernels[k].get("private_segment_fixed_size", 0)}
    assert not used, used


def test_every_instance_of_these_kernels_is_listed(kernels):  # noqa: F811
    prefixes = ("k_xf_long<", "k_xil_long<", "k_yz_long<", "k_y3_fwd_pk<", "k_z3_pk<",
                "k_y3_inv_pk<", "k_small<")
    extra = [k for k in kernels if k.startswith(prefixes) and k not in REACHED]
    assert not extra, extra
