"""Kernels compiled per lmax (and per radial count in the vector pair adjoint):
every lmax in FP32, with the finalisation folded into the pair adjoint and with
the two as kernels of their own, against the oracle.

Tolerance: FP32 rounds at 6e-8; a force sums up to about 1e5 products (the
order-3 contraction at 16 channels), so independent roundings leave 6e-8 x
sqrt(1e5) = 2e-5 of the sum of magnitudes; 3e-5 of the largest force.
"""
import os

import numpy as np
import pytest

import oracle as O
from gen import workloads as W
from tests.gpu_common import rel_force_err, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("n_rad,lmax", [(3, 0), (8, 1), (12, 2), (5, 3), (16, 4), (8, 5), (12, 5), (7, 6), (16, 6)])
def test_fp32_every_lmax(n_rad, lmax, fused):
    w = W.tiny(seed=33, n_rad=n_rad, lmax=lmax)
    w["model"]["ace"]["c3"] *= (4.0 / n_rad) ** 3
    ref = O.mixed(w, O.MODE_ALL_EXPENSIVE)
    print(f"n_rad {n_rad} lmax {lmax} fused {fused}", flush=True)
    if not fused:
        os.environ["MLMIX_FUSE_FIN"] = "0"
    try:
        g = run_gpu(w, O.MODE_ALL_EXPENSIVE, precision="fp32")
    finally:
        os.environ.pop("MLMIX_FUSE_FIN", None)
    assert rel_force_err(g["forces"], ref["forces"]) < 3e-5
    assert np.abs(g["e_exp"] - ref["e_exp"]).max() < 3e-5 * max(1.0, np.abs(ref["e_exp"]).max())
