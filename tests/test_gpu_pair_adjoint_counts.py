"""The vector pair adjoints at every kind of radial count: below, at and above
the multiples of four that they are compiled for, with one to eight species
(the padded rows of the species lie side by side), against the oracle.

Tolerance: FP64 as in the suite (1e-10 of the largest force). FP32 rounds at
6e-8; a force sums up to about 1e5 products, so independent roundings leave
6e-8 x sqrt(1e5) = 2e-5 of the sum of magnitudes; 3e-5 of the largest force.
"""
import numpy as np
import pytest

import oracle as O
from gen import workloads as W
from tests.gpu_common import rel_force_err, run_gpu

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-10, "fp32": 3e-5}


def _cell(ns, n_rad, lmax):
    w = W.tiny(seed=51, n_rad=n_rad, lmax=lmax, order=2)
    r = W._streams(52)
    w["model"]["n_species"] = ns
    w["model"]["ace"] = W.ace_params(r[1], ns, n_rad, lmax, 2, 4.2, W.ACE_SCALE["tiny"])
    w["model"]["uf3"] = W.uf3_params(r[2], ns, 8, 4.2, 4, 3.2)
    w["species"] = np.random.default_rng(5).integers(0, ns, size=len(w["pos"])).astype(np.int32)
    return w


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("ns,n_rad,lmax", [(1, 1, 6), (1, 4, 5), (1, 5, 6), (1, 10, 5), (1, 13, 6), (1, 16, 5),
                                           (2, 3, 5), (2, 5, 5), (2, 9, 2), (3, 2, 6), (3, 7, 3), (8, 1, 6),
                                           (8, 5, 2)])
def test_counts(monkeypatch, ns, n_rad, lmax, prec):
    w = _cell(ns, n_rad, lmax)
    print(f"{prec} ns {ns} n_rad {n_rad} lmax {lmax}", flush=True)
    # FP32: the vector form whatever the size of the system and the model
    monkeypatch.setenv("MLMIX_FUSE_FIN", "0")
    if prec == "fp32" and lmax < 5:
        monkeypatch.setenv("MLMIX_BASIS_MFMA", "0")
    ref = O.mixed(w, O.MODE_ALL_EXPENSIVE)
    g = run_gpu(w, O.MODE_ALL_EXPENSIVE, precision=prec)
    assert rel_force_err(g["forces"], ref["forces"]) < TOL[prec]
    assert np.abs(g["e_exp"] - ref["e_exp"]).max() < TOL[prec] * max(1.0, np.abs(ref["e_exp"]).max())
