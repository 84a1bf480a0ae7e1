"""The wide order-3 contraction of models of several species, whose atoms are
split into those that meet the first species alone and the others: every
padded width, radial counts that are no multiple of 4, all and none of the
atoms in either class, and class sizes on both sides of a 16-atom tile.

Tolerance: FP32 rounds at 6e-8; a force sums up to about 1e5 products, so
independent roundings leave 6e-8 x sqrt(1e5) = 2e-5 of the sum of magnitudes;
3e-5 of the largest force. BF16 rounds both factors of a product at 2e-3: 4e-3
of the sum of magnitudes, which exceeds the largest force by a small factor;
2e-2 of the largest force.
"""
import numpy as np
import pytest

import oracle as O
from gen import workloads as W
from tests.gpu_common import rel_force_err, run_gpu

pytestmark = pytest.mark.gpu
TOL = {"fp32": 3e-5, "bf16": 2e-2}


def _cell(species_of, ns, n_rad, lmax, seed=41):
    w = W.tiny(seed=seed, cells=4, n_rad=n_rad, lmax=lmax)
    r = W._streams(seed + 1)
    w["model"]["n_species"] = ns
    w["model"]["ace"] = W.ace_params(r[1], ns, n_rad, lmax, 3, 4.2, W.ACE_SCALE["tiny"])
    w["model"]["ace"]["c3"] *= (4.0 / n_rad) ** 3
    w["model"]["uf3"] = W.uf3_params(r[2], ns, 8, 4.2, 4, 3.2)
    w["species"] = np.ascontiguousarray(species_of(len(w["pos"])), dtype=np.int32)
    return w


def _one(n):
    s = np.zeros(n)
    s[n // 2] = 1
    return s


def _random(ns):
    return lambda n: np.random.default_rng(5).integers(0, ns, size=n)


def _compare(w, mode):
    ref = O.mixed(w, mode)
    for prec, tol in TOL.items():
        print(f"{prec} |S| {len(ref['S'])}", flush=True)
        g = run_gpu(w, mode, precision=prec)
        assert np.array_equal(g["S"], ref["S"])
        assert rel_force_err(g["forces"], ref["forces"]) < tol
        assert np.abs(g["e_exp"] - ref["e_exp"]).max() < tol * max(1.0, np.abs(ref["e_exp"]).max())


@pytest.mark.parametrize("ns,n_rad,lmax", [(2, 1, 2), (2, 3, 3), (2, 6, 2), (2, 7, 3), (2, 8, 2), (3, 5, 2),
                                           (2, 9, 3), (2, 12, 2), (2, 14, 1), (3, 10, 1), (2, 16, 2), (4, 8, 1)])
def test_widths(ns, n_rad, lmax):
    _compare(_cell(_one, ns, n_rad, lmax), O.MODE_ALL_EXPENSIVE)


@pytest.mark.parametrize("species_of", [np.zeros, np.ones, _random(2)])
def test_one_class(species_of):
    _compare(_cell(species_of, 2, 5, 3), O.MODE_ALL_EXPENSIVE)


@pytest.mark.parametrize("n_s", [1, 15, 16, 17, 33])
def test_tile_edges(n_s):
    w = _cell(_one, 2, 6, 2)
    d = w["pos"] - w["L"] / 2
    d -= w["L"] * np.round(d / w["L"])
    r = np.sort(np.linalg.norm(d, axis=1))
    w["regions"] = [W.sphere(w["L"] / 2, 0.5 * (r[n_s - 1] + r[n_s]) - 0.3, 0.3)]
    w["r_buffer"] = 0.0
    # the other species far from the sphere, then at its centre
    far = np.linalg.norm(d, axis=1)
    for i in (np.argmax(far), np.argmin(far)):
        w["species"] = np.zeros(len(w["pos"]), np.int32)
        w["species"][i] = 1
        _compare(w, O.MODE_MIXED)
