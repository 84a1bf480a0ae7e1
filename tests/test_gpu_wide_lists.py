"""The class lists of the wide order-3 contraction over several workgroups of
1024 S atoms: |S| on both sides of the workgroup's size, capacities with a
workgroup per 1024 atoms and above (65,536), where each takes several rounds, and
more tiles than workgroups. About one atom in a hundred is of
the second species, so both classes hold atoms of every workgroup.

Tolerance against the oracle: FP32 rounds at 6e-8; a force sums up to about 1e4
products (two and six channels, lmax 1), so independent roundings leave 6e-8 x
1e2 = 6e-6 of the sum of magnitudes; 3e-5 of the largest force. The capacity
does not change the order, and so not the bits.
"""
import numpy as np
import pytest

import oracle as O
from gen import workloads as W
from tests.gpu_common import rel_force_err, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _two_classes(monkeypatch):
    """Light models, which would run as one class, in two."""
    monkeypatch.setenv("MLMIX_O3_CLASSES", "1")


def _cell(cells, n_rad, lmax, seed=61):
    w = W.tiny(seed=seed, cells=cells, n_rad=n_rad, lmax=lmax)
    r = W._streams(seed + 1)
    w["model"]["n_species"] = 2
    w["model"]["ace"] = W.ace_params(r[1], 2, n_rad, lmax, 3, 4.2, W.ACE_SCALE["tiny"])
    w["model"]["uf3"] = W.uf3_params(r[2], 2, 8, 4.2, 0, 3.2)
    w["species"] = (np.random.default_rng(6).random(len(w["pos"])) < 0.01).astype(np.int32)
    return w


def _with_s(w, n_s):
    """A sphere that holds n_s atoms, without a buffer."""
    d = w["pos"] - w["L"] / 2
    d -= w["L"] * np.round(d / w["L"])
    r = np.sort(np.linalg.norm(d, axis=1))
    w["regions"] = [W.sphere(w["L"] / 2, 0.5 * (r[n_s - 1] + r[n_s]) - 0.3, 0.3)]
    w["r_buffer"] = 0.0
    return w


def _check(w, mode, s_cap=0, ref=None):
    from paper_2502_19081_amd import core
    model = core.Model(w["model"], precision="fp32")
    _, sy, pos, sp = core.system_for(w, model=model, s_cap=s_cap)
    g = run_gpu(w, mode, system=(sy, pos, sp))
    if ref is not None:
        assert np.array_equal(g["S"], ref["S"])
        assert rel_force_err(g["forces"], ref["forces"]) < 3e-5
        assert np.abs(g["e_exp"] - ref["e_exp"]).max() < 3e-5 * max(1.0, np.abs(ref["e_exp"]).max())
    return g


@pytest.mark.parametrize("n_s", [1023, 1024, 1025, 2049, 3100])
def test_several_workgroups(n_s):
    w = _with_s(_cell(12, 6, 1), n_s)
    print(f"|S| {n_s}", flush=True)
    ref = O.mixed(w, O.MODE_MIXED)
    assert len(_check(w, O.MODE_MIXED, ref=ref)["S"]) == n_s


def test_capacity_does_not_matter():
    w = _with_s(_cell(33, 4, 1), 3100)  # 71,874 atoms
    print("|S| 3100, capacities 71,874 and 4,000", flush=True)
    ref = O.mixed(w, O.MODE_MIXED)
    all_atoms, few = _check(w, O.MODE_MIXED, ref=ref), _check(w, O.MODE_MIXED, s_cap=4000)
    for k in ("forces", "e_exp"):
        assert np.array_equal(all_atoms[k], few[k]), k


def test_several_rounds():
    w = _cell(33, 2, 1)  # two rounds of each workgroup
    print("|S| 71,874", flush=True)
    ref = O.mixed(w, O.MODE_ALL_EXPENSIVE)
    assert len(_check(w, O.MODE_ALL_EXPENSIVE, ref=ref)["S"]) == len(w["pos"])


def _widths(species_of, ns, n_rad, lmax):
    w = W.tiny(seed=71, cells=4, n_rad=n_rad, lmax=lmax)
    r = W._streams(72)
    w["model"]["n_species"] = ns
    w["model"]["ace"] = W.ace_params(r[1], ns, n_rad, lmax, 3, 4.2, W.ACE_SCALE["tiny"])
    w["model"]["uf3"] = W.uf3_params(r[2], ns, 8, 4.2, 0, 3.2)
    g = np.random.default_rng(7)
    n = len(w["pos"])
    w["species"] = {"dilute": (g.random(n) < 0.02).astype(np.int32), "first": np.zeros(n, np.int32),
                    "second": np.ones(n, np.int32),
                    "alloy": g.integers(0, ns, n).astype(np.int32)}[species_of]
    return w


# One class and two give the same bits, whatever the width and the format of the
# operands, and with every split of a tile; and the order-3 term is in them: without
# it nearly every force has other bits.
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("species_of", ["dilute", "first", "second", "alloy"])
@pytest.mark.parametrize("ns,n_rad,lmax", [(2, 1, 2), (2, 3, 3), (2, 6, 2), (2, 7, 3), (3, 5, 2), (2, 9, 3),
                                           (2, 12, 2), (2, 14, 1), (3, 10, 1), (2, 16, 2), (4, 8, 1)])
def test_one_class_and_two(monkeypatch, prec, species_of, ns, n_rad, lmax):
    w = _widths(species_of, ns, n_rad, lmax)
    print(f"{prec} {species_of} {ns} x {n_rad}, lmax {lmax}", flush=True)

    def run(classes, split=None):
        monkeypatch.setenv("MLMIX_O3_CLASSES", classes)
        if split:
            monkeypatch.setenv("MLMIX_O3_MAX_SPLIT", split)
        return run_gpu(w, O.MODE_ALL_EXPENSIVE, precision=prec)

    one = run("0")
    for got in (run("1"), run("1", "1"), run("1", "2")):
        for k in ("forces", "e_exp"):
            assert np.array_equal(one[k], got[k]), k
    w["model"]["ace"]["c3"] = np.zeros_like(w["model"]["ace"]["c3"])
    assert (run("1")["forces"] != one["forces"]).mean() > 0.9
