"""Sizes at which the fit's kernels change their shape: no 3-body term, both
3-body widths, long 2-body records (fewer per batch), many species pairs (more
than one column tile); parameter and hard-row counts on both sides of the
search's panels, wavefronts and row tiles.

Tolerances: design rows sum at most a few hundred products of numbers of order
one, so 1e-12 of the largest entry as in the other design tests; the search's
solutions may lose n_params x condition x 1.1e-16 of the largest coefficient
each way. With more hard rows than parameters alpha may be out of reach: both
then return the solution of the smallest residual seen, which is flat in lambda,
so the residuals are compared and not lambda.
"""
import numpy as np
import pytest

from gen import workloads as W
from oracle import fit as OF
from tests.test_gpu_fit import _design_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_species,nk2,nk3", [(1, 8, 0), (1, 4, 4), (1, 17, 5), (1, 64, 4), (2, 9, 4), (3, 12, 0), (2, 13, 0)])
def test_design_shapes(n_species, nk2, nk3):
    r = np.random.default_rng(5)
    w = W.tiny(seed=41, sigma=0.15)
    w["species"] = r.integers(0, n_species, len(w["pos"])).astype(np.int32)
    m = dict(w["model"], n_species=n_species, uf3=W.uf3_params(r, n_species, nk2, 4.2, nk3, 3.2),
             ace=W.ace_params(r, n_species, 2, 1, 2, 4.2, (1.0, 1.0, 0.0)))
    print(f"design {n_species} species, knots {nk2} {nk3}", flush=True)
    A, fit = _design_gpu(m, dict(pos=w["pos"], L=w["L"], periodic=w["periodic"]), w["species"])
    ref = OF.design(m, w["pos"], w["species"], w["L"], w["periodic"])
    assert A.shape == ref.shape
    assert np.abs(A - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("nd,nh", [(1, 1), (7, 17), (15, 4), (16, 16), (17, 65), (48, 3), (63, 10), (64, 64), (65, 33),
                                   (81, 102), (112, 5), (120, 130)])
def test_search_sizes(nd, nh):
    import torch
    from gen import fitdata as FD
    from paper_2502_19081_amd import core
    from paper_2502_19081_amd.fit import CheapFit
    r = np.random.default_rng(100 * nd + nh)
    S = r.normal(size=(4 * nd + 40, nd))
    G, b = S.T @ S, r.normal(size=nd) * nd
    AH, yH = r.normal(size=(nh, nd)), r.normal(size=nh)
    wH = r.uniform(0.5, 2.0, nh)
    free = OF.solve_fixed(G, b, np.zeros_like(G), np.zeros(nd), 0.0, 1e-3)
    alpha = 0.3 * OF.hard_residual(AH, yH, free, wH)
    print(f"search nd {nd} nh {nh}", flush=True)
    c, info = OF.constrained_fit(G, b, AH, yH, alpha, lam0=1e-3, ridge=1e-3, wH=wH)
    fit = CheapFit(core.Model(FD.fit_model(), precision="fp64"))
    fit.nd = nd
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    u, got = fit.constrained(t(G), t(b), t(AH), t(yH), alpha, lam0=1e-3, ridge=1e-3, wH=t(wH))
    assert got["status"] == info["status"] and got["n_solves"] == info["n_solves"]
    cond = np.linalg.cond(G + info["lam"] * (AH.T @ (wH[:, None] * AH)) + 1e-3 * np.eye(nd))
    tol = max(2 * nd * cond * 1.1e-16, 1e-13)
    if info["status"] == 1:
        assert abs(got["residual"] - info["residual"]) <= tol * info["residual"]
        return
    assert abs(got["lam"] - info["lam"]) <= 1e-12 * info["lam"]
    assert np.abs(u.cpu().numpy() - c).max() <= tol * np.abs(c).max()
