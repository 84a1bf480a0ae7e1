"""The FP64 order-3 contraction on the matrix cores (one species, at most 16
channels) against the oracle at the edges of its tiles: channel counts on both
sides of every padded width (4, 8, 12, 16), every lmax, and |S| on both sides of
the 16-atom tile.

Tolerance: an output of the contraction is a sum of at most about 1e5 products
(channel pairs x Gaunt entries x blocks of one l3), so its rounding is below
1e5 x 1.1e-16 = 1.1e-11 of the sum of the magnitudes; 1e-10 of the largest
force or energy leaves the usual factor for cancellation (the suite's FP64
bound).
"""
import numpy as np
import pytest

from gen import workloads as W
from tests.test_gpu_parity import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rad,lmax", [(1, 1), (3, 0), (4, 2), (5, 3), (8, 4), (9, 1), (11, 3), (12, 4),
                                        (13, 2), (16, 3), (14, 5), (16, 6)])
def test_channels_and_lmax(n_rad, lmax):
    w = W.tiny(seed=31, n_rad=n_rad, lmax=lmax)
    w["model"]["ace"]["c3"] *= (4.0 / n_rad) ** 3
    _check(w, "all_expensive", "fp64")


@pytest.mark.parametrize("n_s", [1, 15, 16, 17, 32, 33])
def test_tile_edges(n_s):
    w = W.tiny(seed=32, n_rad=6, lmax=3)
    d = w["pos"] - w["L"] / 2
    d -= w["L"] * np.round(d / w["L"])
    r = np.sort(np.linalg.norm(d, axis=1))
    w["regions"] = [W.sphere(w["L"] / 2, 0.5 * (r[n_s - 1] + r[n_s]) - 0.3, 0.3)]
    w["r_buffer"] = 0.0
    g, _ = _check(w, "mixed", "fp64")
    assert len(g["S"]) == n_s
