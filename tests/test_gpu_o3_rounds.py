"""Order-3 contractions with more tiles of 16 S atoms than workgroups, so that a
workgroup takes several: FP64 (at most 512 workgroups, 1,158 tiles) and the wide
form as one class, against the oracle.

Tolerance: FP64 as in the suite (1e-10 of the largest force). FP32 rounds at
6e-8; a force sums up to about 1e4 products (at most six channels, lmax 1), so
independent roundings leave 6e-6 of the sum of magnitudes; 3e-5 of the largest.
"""
import numpy as np
import pytest

import oracle as O
from gen import workloads as W
from tests.gpu_common import rel_force_err, run_gpu
from tests.test_gpu_wide_lists import _cell

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32": 3e-5}


@pytest.mark.parametrize("prec,ns,n_rad", [("fp64", 1, 3), ("fp64", 1, 6), ("fp32", 2, 2)])
def test_more_tiles_than_workgroups(prec, ns, n_rad):
    w = _cell(21, n_rad, 1) if ns == 2 else W.tiny(seed=81, cells=21, n_rad=n_rad, lmax=1)
    print(f"{prec} {ns} x {n_rad}, |S| {len(w['pos'])}", flush=True)
    ref = O.mixed(w, O.MODE_ALL_EXPENSIVE)
    g = run_gpu(w, O.MODE_ALL_EXPENSIVE, precision=prec)
    assert np.array_equal(g["S"], ref["S"])
    assert rel_force_err(g["forces"], ref["forces"]) < TOL[prec]
    assert np.abs(g["e_exp"] - ref["e_exp"]).max() < TOL[prec] * max(1.0, np.abs(ref["e_exp"]).max())
