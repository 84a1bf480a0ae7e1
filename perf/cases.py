"""Performance cases of the mixed force evaluation: what a user of this package
has it do, from a single force call on a few hundred atoms to molecular
dynamics of a million, and the constrained fit of the cheap potential.

Every case is one of five kinds of call:
  force  System.compute: one force call (a relaxation, a NEB image, a label)
  md     a short MD run: System.compute, then System.vv_steps
  batch  several replicas in one Batch: Batch.compute, then Batch.vv_steps
  grad   site energies and their position gradient through torch.autograd
  fit    design rows, normal equations and the lambda search of CheapFit

The atoms are displaced bcc W (a = 3.165 A), the potentials random linear
coefficients of the shapes that the tests and the benchmark use. Nothing here
calls the package except prepare() and run(); exact() evaluates the same
definitions with plain torch in 64 bits.

Sizes in a case: cells (conventional bcc cells along x, y, z), vacancies
(random sites left out), sigma (displacement, A); potential names one of
POTENTIALS; regions is where lambda > 0: "sphere" (one 8 + 2 A sphere in the
middle), "vacancies" (7 + 2 A at every vacancy), "cylinder" (12 + 3 A about
the z axis, with free surfaces along x and y).
"""
import math

import numpy as np
import torch

from paper_2502_19081_amd import binding, core
from paper_2502_19081_amd.autograd import expensive_energy
from paper_2502_19081_amd.fit import CheapFit

DEV = "cuda"
A_W = 3.165
KAPPA = 9.648533212e-3
KB = 8.617333262e-5
MASS = (183.84, 4.002602)
FREE = 12.0  # vacuum beside a free surface, A
MODES = {"mixed": binding.MODE_MIXED, "expensive": binding.MODE_ALL_EXPENSIVE,
         "cheap": binding.MODE_ALL_CHEAP}

# species, (radial functions, lmax, order, cutoff), scale of the coefficients
# per order, 2-body (knots, cutoff), 3-body (knots, cutoff), buffer radius
POTENTIALS = {
    "pair": (1, (8, 3, 2, 5.0), (0.6, 0.3, 0.0), (12, 5.0), (0, 3.5), 5.0),
    "w": (1, (12, 4, 3, 5.5), (0.2, 0.02, 0.01), (16, 5.5), (6, 3.5), 5.5),
    "wide": (1, (16, 5, 3, 5.0), (0.3, 0.008, 0.017), (16, 5.5), (6, 3.5), 5.0),
    "whe": (2, (12, 4, 3, 5.0), (0.025, 0.0075, 0.003), (16, 6.0), (6, 3.5), 5.0),
}


def _single(name, kind, cells, potential, precision, mode="mixed", regions="sphere", vacancies=0,
            sigma=0.08, rebuild=True, steps=0, cubic=False, masked=False):
    c = dict(name=name, kind=kind, nx=cells[0], ny=cells[1], nz=cells[2], vacancies=vacancies,
             sigma=sigma, potential=potential, precision=precision, mode=mode, regions=regions,
             rebuild=rebuild, steps=steps, cubic=cubic, masked=masked)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # the smallest call: one vacancy in 5^3 cells, the verification precision
        _single("force_fp64_249", "force", (5, 5, 5), "pair", "fp64", vacancies=1, sigma=0.05),
        # one relaxation step of a ragged cell, cubic blend, the cheap potential masked
        _single("force_fp32_1977", "force", (9, 11, 10), "w", "fp32", vacancies=3,
                rebuild=False, cubic=True, masked=True),
        # a label for fitting: the expensive potential on every atom, FP64
        _single("label_fp64_2000", "force", (10, 10, 10), "w", "fp64", mode="expensive"),
        # the all-expensive reference run that a mixed run is compared with
        _single("expensive_fp32_8192", "force", (16, 16, 16), "w", "fp32", mode="expensive"),
        # the paper's usual cell size: mixed MD about one defect
        _single("md_fp32_8191", "md", (16, 16, 16), "w", "fp32", vacancies=1, steps=20),
        # a screw-dislocation sized column: free surfaces, a cylinder along the line
        _single("md_fp32_54000", "md", (30, 30, 30), "w", "fp32", regions="cylinder", steps=10),
        # many defects in a large cell, BF16 operands in the order-3 contraction
        _single("md_bf16_249960", "md", (50, 50, 50), "wide", "bf16", regions="vacancies",
                vacancies=40, sigma=0.05, steps=4),
        # the largest cell: 200 vacancies in 80^3 cells
        _single("md_fp32_1023800", "md", (80, 80, 80), "wide", "fp32", regions="vacancies",
                vacancies=200, sigma=0.05, steps=4),
        # serving: He impact replicas of 2,000 to 20,000 atoms in one batch, as many
        # as run together at ordinary load, and a fuller batch
        dict(name="batch_bf16_5", kind="batch", replicas=5, smallest=2000, largest=20000,
             precision="bf16", steps=10),
        dict(name="batch_fp32_16", kind="batch", replicas=16, smallest=2000, largest=20000,
             precision="fp32", steps=5),
        # site energies and their gradient under autograd
        _single("grad_fp64_1024", "grad", (8, 8, 8), "w", "fp64", mode="expensive"),
        # the constrained fit: snapshots of a 2,000-atom cell and 102 strained cells
        dict(name="fit_20x2000", kind="fit", snapshots=20, cells=10, strained=102,
             strained_cells=5, knots2=12, knots3=5, sigma=0.1),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("force", "force", "md", "md", "batch", "grad", "fit"))
    if kind == "batch":
        return dict(kind="batch", replicas=log(2, 16), smallest=2000,
                    largest=log(3000, 20000), precision=rng.choice(("fp32", "bf16")),
                    steps=rng.randint(2, 8))
    if kind == "fit":
        return dict(kind="fit", snapshots=rng.randint(2, 20), cells=rng.randint(5, 10),
                    strained=rng.randint(10, 102), strained_cells=5, knots2=rng.randint(8, 16),
                    knots3=rng.choice((0, 4, 5)), sigma=0.1)
    precision = rng.choice(("fp32", "fp32", "bf16", "fp64"))
    if kind == "grad":
        potential, mode = "w", rng.choice(("mixed", "expensive"))
    else:
        potential = rng.choice(("w", "wide")) if precision == "bf16" else \
            rng.choice(("pair", "w", "wide"))
        mode = rng.choice(("mixed", "mixed", "mixed", "expensive", "cheap"))
    # the side of a cell of the case's atoms; FP64 and all-expensive calls are small ones
    most = 120000 if mode != "expensive" else 16000
    most = min(most, {"fp64": 3000, "fp32": 120000, "bf16": 120000}[precision])
    side = (log(300, most) / 2.0) ** (1.0 / 3.0)
    cells = [max(5, int(round(side * rng.uniform(0.85, 1.2)))) for _ in range(3)]
    regions = rng.choice(("sphere", "sphere", "vacancies", "cylinder"))
    vacancies = rng.randint(1, max(1, min(20, cells[0] * cells[1] * cells[2] // 400)))
    return _single(None, kind, cells, potential, precision, mode=mode, regions=regions,
                   vacancies=vacancies, sigma=rng.uniform(0.03, 0.1),
                   rebuild=rng.random() < 0.7, steps=rng.randint(2, 12) if kind == "md" else 0,
                   cubic=rng.random() < 0.3,
                   masked=mode == "mixed" and kind != "grad" and rng.random() < 0.2)


# ------------------------------------------------------------------ inputs

def _potential(name, seed, knots2=None, knots3=None):
    """Random coefficients in the layout that core.Model takes."""
    ns, (n_rad, lmax, order, rcut), scale, (k2, rc2), (k3, rc3), _ = POTENTIALS[name]
    if knots2 is not None:
        k2, k3 = knots2, knots3
    r = np.random.default_rng([seed, 11])
    nchan, L1 = ns * n_rad, lmax + 1
    K = nchan * L1
    weak = 0.05 if ns > 1 else 1.0
    ace = dict(n_rad=n_rad, lmax=lmax, order=order, rcut=rcut, c0=r.normal(size=ns),
               c1=r.normal(size=(ns, nchan)) * scale[0],
               c2=r.normal(size=(ns, L1, nchan, nchan)) * scale[1],
               c3=r.normal(size=(ns, K, K, K)) * scale[2] if order >= 3 else np.zeros((ns, 1, 1, 1)))
    c2 = r.normal(size=(ns, ns, k2 + 2)) * 0.1 * weak
    c2 = 0.5 * (c2 + c2.transpose(1, 0, 2))
    c2[:, :, -3:] = 0.0
    c3 = np.zeros((ns, 1, 1, 1))
    if k3:
        nb = k3 + 2
        c3 = r.normal(size=(ns, nb, nb, nb)) * 0.02 * weak
        c3 = 0.5 * (c3 + c3.transpose(0, 2, 1, 3))
        c3[:, -3:] = 0.0
        c3[:, :, -3:] = 0.0
    if ns > 1:  # a smooth He-W repulsion in both potentials
        ace["c1"][0, n_rad] = ace["c1"][1, 0] = 100.0
        ramp = np.maximum(0.0, 1.0 - np.arange(k2 + 2) / 7.0) ** 2 * 20.0
        ramp[-3:] = 0.0
        c2[0, 1] += ramp
        c2[1, 0] += ramp
    return dict(n_species=ns, skin=1.0, ace=ace,
                uf3=dict(n_knots2=k2, rcut2=rc2, c2=c2, n_knots3=k3, rcut3=rc3, c3=c3))


def _lattice(nx, ny, nz):
    g = torch.meshgrid(*(torch.arange(m, device=DEV, dtype=torch.float64) for m in (nx, ny, nz)),
                       indexing="ij")
    corner = torch.stack([x.reshape(-1) for x in g], 1)
    return torch.stack([corner, corner + 0.5], 1).reshape(-1, 3) * A_W


def _wrap(pos, L, periodic):
    """(3, n) positions into [0, L) along periodic dimensions."""
    for k in range(3):
        if periodic[k]:
            pos[k] -= L[k] * torch.floor(pos[k] / L[k])
            pos[k][pos[k] >= L[k]] = 0.0
    return pos


def _velocities(mass, T, gen):
    v = torch.randn(3, len(mass), generator=gen, device=DEV, dtype=torch.float64)
    v *= torch.sqrt(KAPPA * KB * T / mass)
    return v - (v * mass).sum(1, keepdim=True) / mass.sum()


def _atoms(case, seed):
    gen = torch.Generator(DEV).manual_seed(seed)
    rng = np.random.default_rng([seed, 7])
    pos = _lattice(case["nx"], case["ny"], case["nz"])
    L = [case[k] * A_W for k in ("nx", "ny", "nz")]
    periodic = [1, 1, 1]
    gone = np.sort(rng.choice(len(pos), size=case["vacancies"], replace=False))
    holes = pos[torch.from_numpy(gone).to(DEV)].cpu().numpy()
    keep = torch.ones(len(pos), dtype=torch.bool, device=DEV)
    keep[torch.from_numpy(gone).to(DEV)] = False
    pos = pos[keep]
    pos = (pos + torch.randn(pos.shape, generator=gen, device=DEV, dtype=torch.float64)
           * case["sigma"]).t().contiguous()
    if case["regions"] == "cylinder":
        periodic = [0, 0, 1]
        pos[:2] += FREE
        L = [L[0] + 2 * FREE, L[1] + 2 * FREE, L[2]]
    blend = int(case["cubic"])
    middle = [x / 2 for x in L]
    if case["regions"] == "cylinder":
        regions = [dict(type=1, axis=2, center=middle, r_core=12.0, r_blend=3.0, blend=blend)]
    elif case["regions"] == "vacancies":
        regions = [dict(type=0, center=[float(x) for x in h], r_core=7.0, r_blend=2.0, blend=blend)
                   for h in holes]
    else:
        regions = [dict(type=0, center=middle, r_core=8.0, r_blend=2.0, blend=blend)]
    n = pos.shape[1]
    mass = torch.full((n,), MASS[0], device=DEV, dtype=torch.float64)
    return dict(n=n, pos=_wrap(pos, L, periodic), species=torch.zeros(n, dtype=torch.int32, device=DEV),
                mass=mass, vel=_velocities(mass, 300.0, gen), L=L, periodic=periodic,
                regions=regions, weights=torch.randn(n, generator=gen, device=DEV, dtype=torch.float64))


def _replicas(case, seed):
    """W(001) slabs with one 10-80 eV He atom above the surface each; sizes
    spread evenly over the logarithm of the range."""
    gen = torch.Generator(DEV).manual_seed(seed)
    rng = np.random.default_rng([seed, 5])
    out = []
    for k in range(case["replicas"]):
        f = (k + 0.5) / case["replicas"]
        target = case["smallest"] * (case["largest"] / case["smallest"]) ** f
        m = max(2, int(round(target / 392.0)))
        pos = _lattice(14, 14, m)
        pos = pos + 0.02 * torch.randn(pos.shape, generator=gen, device=DEV, dtype=torch.float64)
        pos[:, 2] += 20.0
        top = 20.0 + (m - 0.5) * A_W
        edge = 14 * A_W
        he = torch.tensor([[rng.uniform(0, edge), rng.uniform(0, edge), top + rng.uniform(1.5, 6.0)]],
                          device=DEV, dtype=torch.float64)
        pos = torch.cat([pos, he]).t().contiguous()
        n = pos.shape[1]
        L, periodic = [edge, edge, top + 300.0], [1, 1, 0]
        species = torch.zeros(n, dtype=torch.int32, device=DEV)
        species[-1] = 1
        mass = torch.where(species == 1, MASS[1], MASS[0]).to(torch.float64)
        vel = _velocities(mass, 1000.0, gen)
        speed = math.sqrt(2.0 * rng.uniform(10.0, 80.0) * KAPPA / MASS[1])
        vel[:, -1] = torch.tensor([0.0, 0.0, -speed], dtype=torch.float64)
        out.append(dict(n=n, pos=_wrap(pos, L, periodic), vel=vel, mass=mass, species=species, L=L,
                        periodic=periodic, regions=[dict(type=0, center=[0.0] * 3, r_core=6.0,
                                                         r_blend=2.0, follow_atom=n - 1)]))
    return out


def _configurations(case, seed):
    """Fit data: thermal snapshots, and cells strained along x, with the
    energies and forces of a Morse solid as labels."""
    gen = torch.Generator(DEV).manual_seed(seed)
    out = []
    base = _lattice(case["cells"], case["cells"], case["cells"]).t().contiguous()
    for _ in range(case["snapshots"]):
        L = [case["cells"] * A_W] * 3
        x = base + case["sigma"] * torch.randn(base.shape, generator=gen, device=DEV, dtype=torch.float64)
        out.append(dict(pos=_wrap(x, L, [1, 1, 1]), L=L, hard=False))
    m = case["strained_cells"]
    base = _lattice(m, m, m).t().contiguous()
    small = 0.01 * torch.randn(base.shape, generator=gen, device=DEV, dtype=torch.float64)
    for k in range(case["strained"]):
        e = 0.01 * (k + 0.5) / case["strained"] - 0.005
        L = [m * A_W * (1.0 + e), m * A_W, m * A_W]
        x = base + small
        x = x * torch.tensor([[1.0 + e], [1.0], [1.0]], device=DEV, dtype=torch.float64)
        out.append(dict(pos=_wrap(x, L, [1, 1, 1]), L=L, hard=True))
    for c in out:
        n = c["pos"].shape[1]
        i, j, d = _pairs(c["pos"], c["L"], [1, 1, 1], 5.5)
        r = d.norm(dim=1)
        x = torch.exp(-1.4 * (r - 2.8))
        cut = (1.0 - (r / 5.5) ** 2) ** 2
        phi = x * (x - 2.0)
        dphi = -1.4 * x * (2.0 * x - 2.0) * cut + phi * 2.0 * (1.0 - (r / 5.5) ** 2) * (-2.0 * r / 5.5 ** 2)
        c["n"], c["energy"] = n, 0.25 * (phi * cut).sum().reshape(1)
        g = 0.25 * (dphi / r)[:, None] * d
        f = torch.zeros(n, 3, device=DEV, dtype=torch.float64).index_add_(0, i, g).index_add_(0, j, -g)
        c["forces"] = f.t().contiguous()
    return out


def _fit_data(case, seed):
    cfg = _configurations(case, seed)
    soft, hard = [c for c in cfg if not c["hard"]], [c for c in cfg if c["hard"]]
    y = torch.cat([torch.cat([c["energy"], c["forces"].reshape(-1)]) for c in soft])
    w = torch.cat([torch.cat([torch.full((1,), 1.0 / c["n"] ** 2, device=DEV, dtype=torch.float64),
                              torch.ones(3 * c["n"], device=DEV, dtype=torch.float64)]) for c in soft])
    yH = torch.cat([c["energy"] for c in hard])
    wH = torch.tensor([1.0 / c["n"] ** 2 for c in hard], device=DEV, dtype=torch.float64)
    return soft, hard, y, w, yH, wH


# The fit's search: the ridge keeps the normal equations well conditioned, the
# bound on the hard residual (eV per atom, squared, summed) takes a few decades
# of lambda and some bisections.
RIDGE, ALPHA, LAMBDA0 = 1.0, 2e-5, 1e-3


# ---------------------------------------------------------------- prepare, run

def _system(case, a, seed):
    model = core.Model(_potential(case["potential"], seed), precision=case["precision"])
    s_cap = a["n"] // 4 if a["n"] > 200000 else 0
    sy = core.System(model, a["n"], a["L"], a["periodic"], s_cap=s_cap)
    sy.set_regions(a["regions"])
    return sy


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("force", "md", "grad"):
        a = _atoms(case, seed)
        sy = _system(case, a, seed)
        s = dict(kind=kind, case=case, sy=sy, buffer=POTENTIALS[case["potential"]][5],
                 mode=MODES[case["mode"]], **a)
        if kind == "md":
            s["x"], s["v"] = a["pos"].clone(), a["vel"].clone()
        return s
    if kind == "batch":
        r = _replicas(case, seed)
        b = core.Batch(core.Model(_potential("whe", seed), precision=case["precision"]), r)
        s = {k: torch.cat([x[k] for x in r], -1).contiguous()
             for k in ("pos", "vel", "mass", "species")}
        return dict(kind=kind, case=case, batch=b, x=s["pos"].clone(), v=s["vel"].clone(), **s)
    model = core.Model(_potential("w", seed, case["knots2"], case["knots3"]), precision="fp64")
    fit = CheapFit(model)
    soft, hard, y, w, yH, wH = _fit_data(case, seed)

    def items(cfgs):
        offs = np.cumsum([0] + [1 + 3 * c["n"] for c in cfgs])
        rows = torch.empty(int(offs[-1]), fit.nd, dtype=torch.float64, device=DEV)
        out = []
        for c, o in zip(cfgs, offs):
            sy = core.System(model, c["n"], c["L"], [1, 1, 1])
            sp = torch.zeros(c["n"], dtype=torch.int32, device=DEV)
            sy.compute(c["pos"], sp, mode=binding.MODE_ALL_CHEAP, force_rebuild=True)
            out.append((sy, c["pos"], sp, rows[o:o + 1 + 3 * c["n"]]))
        return out, rows, torch.from_numpy(offs[:-1].astype(np.int64)).to(DEV)

    si, rows, _ = items(soft)
    hi, hrows, at = items(hard)
    return dict(kind=kind, case=case, fit=fit, items=si + hi, rows=rows, hrows=hrows, at=at, y=y, w=w,
                yH=yH, wH=wH)


def run(state):
    s, case = state, state["case"]
    if s["kind"] == "force":
        return s["sy"].compute(s["pos"], s["species"], r_buffer=s["buffer"], mode=s["mode"],
                               force_rebuild=case["rebuild"], cheap_masked=case["masked"])
    if s["kind"] == "md":
        sy = s["sy"]
        s["x"].copy_(s["pos"])
        s["v"].copy_(s["vel"])
        how = dict(r_buffer=s["buffer"], mode=s["mode"], cheap_masked=case["masked"])
        out = sy.compute(s["x"], s["species"], force_rebuild=case["rebuild"], **how)
        e = sy.vv_steps(s["x"], s["v"], s["mass"], s["species"], 1.0, case["steps"], **how)
        return dict(out, pos=s["x"], vel=s["v"], energies=e)
    if s["kind"] == "batch":
        b = s["batch"]
        s["x"].copy_(s["pos"])
        s["v"].copy_(s["vel"])
        out = b.compute(s["x"], s["species"], r_buffer=5.0, force_rebuild=True)
        e = b.vv_steps(s["x"], s["v"], s["mass"], s["species"], 0.2, case["steps"], r_buffer=5.0)
        return dict(out, pos=s["x"], vel=s["v"], energies=e)
    if s["kind"] == "grad":
        x = s["pos"].detach().requires_grad_(True)
        e = expensive_energy(x, s["sy"], s["species"], s["buffer"], s["mode"])
        (g,) = torch.autograd.grad(e, x, s["weights"])
        return dict(e=e.detach(), grad=g)
    s["fit"].design_many(s["items"])
    AH = s["hrows"].index_select(0, s["at"])
    G, b = s["fit"].gram(s["rows"], s["y"], s["w"])
    u, info = s["fit"].constrained(G, b, AH, s["yH"], ALPHA, lam0=LAMBDA0, ridge=RIDGE, wH=s["wH"])
    return dict(rows=s["rows"], AH=AH, G=G, b=b, u=u, info=info)


# ------------------------------------------------------------------------ work

def _contraction_flops(n_chan, lmax):
    """Order-3 energy and its derivative by A as one symmetric cubic form:
    for every l1 <= l2 <= l3 the nonzero couplings on the channel pairs, then
    the channel contraction."""
    G = _gaunt(lmax, "cpu")
    f = 0.0
    for l1, l2, l3 in _triples(lmax):
        if l1 <= l2 <= l3:
            nnz = int((_block(G, l1, l2, l3).abs() > 1e-12).sum())
            f += 2 * n_chan ** 2 * nnz + 2 * n_chan ** 3 * (2 * l3 + 1)
    return f


def _call_work(potential, n, n_S, n_cheap):
    """One force call: the flops of both potentials, and its inputs and outputs."""
    ns, (n_rad, lmax, order, rcut), _, (_, rc2), (k3, _), _ = POTENTIALS[potential]
    rho = 2.0 / A_W ** 3
    L2 = (lmax + 1) ** 2
    pe, p2 = (4.0 / 3.0 * math.pi * r ** 3 * rho for r in (rcut, rc2))
    site = pe * (47 + 16 * n_rad + 32 * L2 + 6 * n_rad * L2) + ns * n_rad * L2 * (2 * ns * n_rad + 9)
    if order >= 3:
        site += _contraction_flops(ns * n_rad, lmax)
    cheap = 96 * p2 + (444 * 91 if k3 else 0)
    return n * (24 + 4 + 24 + 24 + 1), n_S * site + n_cheap * cheap


def _n_S(case, n):
    if case["mode"] != "mixed":
        return n if case["mode"] == "expensive" else 0
    rho, buf = 2.0 / A_W ** 3, POTENTIALS[case["potential"]][5]
    if case["regions"] == "cylinder":
        return min(n, math.pi * (15.0 + buf) ** 2 * case["nz"] * A_W * rho)
    if case["regions"] == "vacancies":
        return min(n, case["vacancies"] * 4.0 / 3.0 * math.pi * (9.0 + buf) ** 3 * rho)
    return min(n, 4.0 / 3.0 * math.pi * (10.0 + buf) ** 3 * rho)


def work(case):
    kind = case["kind"]
    if kind == "fit":
        k2, k3 = case["knots2"], case["knots3"]
        cols3 = (k3 - 1) * k3 // 2 * (k3 + 2) if k3 else 0
        nd = k2 - 1 + cols3
        n = case["snapshots"] * 2 * case["cells"] ** 3
        nh = case["strained"] * 2 * case["strained_cells"] ** 3
        # the nonzero products of a triplet on its three atoms, and of a pair
        per_atom = 44 * 4 * 8 + (91 * 64 * 3 * 3 * 2 if k3 else 0)
        rows = 3 * n + case["snapshots"]
        return dict(bytes=24 * (n + nh) + 8 * nd * rows + 8 * nd * case["strained"],
                    flops=(n + nh) * per_atom + rows * nd * (nd + 2))
    if kind == "batch":
        f = [(k + 0.5) / case["replicas"] for k in range(case["replicas"])]
        n = sum(392 * max(2, round(case["smallest"] * (case["largest"] / case["smallest"]) ** x / 392.0))
                for x in f)
        b, fl = _call_work("whe", n, 400 * case["replicas"], n)
        return dict(bytes=(case["steps"] + 1) * b + case["steps"] * 104 * n, flops=(case["steps"] + 1) * fl)
    n = 2 * case["nx"] * case["ny"] * case["nz"] - case["vacancies"]
    if kind == "grad":
        b, f = _call_work(case["potential"], n, _n_S(case, n), 0)
        return dict(bytes=b, flops=f)
    b, f = _call_work(case["potential"], n, _n_S(case, n), 0 if case["mode"] == "expensive" else n)
    return dict(bytes=(case["steps"] + 1) * b + case["steps"] * 104 * n, flops=(case["steps"] + 1) * f)


# ----------------------------------------------------- the same in plain torch

def _fold(d, L, periodic):
    for k in range(3):
        if periodic[k]:
            d[k] = d[k] - L[k] * torch.round(d[k] / L[k])
    return d


def _pairs(pos, L, periodic, rc):
    """Directed pairs (i, j, x_j - x_i) closer than rc, by i. Rows of atoms
    sorted along the longest edge meet only the candidates in reach."""
    n = pos.shape[1]
    ax = max(range(3), key=lambda k: L[k])
    order = torch.argsort(pos[ax])
    p = pos[:, order].contiguous()
    reach = torch.stack([p[ax] - rc, p[ax] + rc])
    shift = [-L[ax], 0.0, L[ax]] if periodic[ax] and L[ax] > 2 * rc else [0.0]
    whole = periodic[ax] and L[ax] <= 2 * rc
    got, step = [], max(64, min(2048, int(4e7 / max(n, 1))))
    for a in range(0, n, step):
        b = min(n, a + step)
        if whole:
            cand = torch.arange(n, device=pos.device)
        else:
            ends = torch.stack([torch.searchsorted(p[ax].contiguous(), torch.stack(
                [reach[0, a] + s, reach[1, b - 1] + s])) for s in shift]).tolist()
            cand = torch.cat([torch.arange(lo, hi, device=pos.device) for lo, hi in ends]).unique()
        d = _fold([p[k, cand][None, :] - p[k, a:b, None] for k in range(3)], L, periodic)
        r2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
        near = r2 < rc * rc
        near[torch.arange(a, b, device=pos.device)[:, None] == cand[None, :]] = False
        i, j = near.nonzero(as_tuple=True)
        got.append((order[i + a], order[cand[j]], torch.stack([x[i, j] for x in d], 1)))
    i, j, d = (torch.cat(x) for x in zip(*got))
    by = torch.argsort(i * n + j)
    return i[by], j[by], d[by]


def _ylm(lmax, u):
    """Real orthonormal spherical harmonics of unit vectors, l^2 + l + m."""
    x, y, z = u.unbind(1)
    c, s = [torch.ones_like(x)], [torch.zeros_like(x)]
    for m in range(lmax):
        c, s = c + [c[m] * x - s[m] * y], s + [s[m] * x + c[m] * y]
    out = []
    for l in range(lmax + 1):
        for m in range(-l, l + 1):
            k = abs(m)
            q = torch.zeros_like(z)
            for t in range((l - k) // 2 + 1):
                f = math.factorial
                v = (-1) ** t * f(2 * l - 2 * t) / (2 ** l * f(t) * f(l - t) * f(l - 2 * t - k))
                q = q + v * z ** (l - 2 * t - k)
            norm = math.sqrt((2 * l + 1) / (4 * math.pi) * math.factorial(l - k) / math.factorial(l + k))
            out.append(norm * q * (1.0 if m == 0 else math.sqrt(2.0) * (c[k] if m > 0 else s[k])))
    return torch.stack(out, 1)


def _gaunt(lmax, device):
    """Integrals of three real harmonics: Gauss-Legendre times the uniform rule."""
    zx, zw = np.polynomial.legendre.leggauss(2 * lmax + 2)
    phi = 2 * np.pi * np.arange(4 * lmax + 4) / (4 * lmax + 4)
    z, f = [a.reshape(-1) for a in np.meshgrid(zx, phi, indexing="ij")]
    w = np.repeat(zw, len(phi)) * 2 * np.pi / len(phi)
    st = np.sqrt(1 - z * z)
    Y = _ylm(lmax, torch.from_numpy(np.stack([st * np.cos(f), st * np.sin(f), z], 1))).numpy()
    return torch.from_numpy(np.einsum("t,ta,tb,tc->abc", w, Y, Y, Y, optimize=True)).to(device)


def _triples(lmax):
    r = range(lmax + 1)
    return [(a, b, c) for a in r for b in r for c in r
            if (a + b + c) % 2 == 0 and abs(a - b) <= c <= a + b]


def _block(G, l1, l2, l3):
    return G[l1 * l1:(l1 + 1) ** 2, l2 * l2:(l2 + 1) ** 2, l3 * l3:(l3 + 1) ** 2]


class _Exact:
    """Both potentials in 64 bits."""

    def __init__(self, pot):
        self.ns, a, u = pot["n_species"], pot["ace"], pot["uf3"]
        self.a, self.u = a, u
        t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)  # noqa: E731
        self.c0, self.c1, self.c2 = t(a["c0"]), t(a["c1"]), t(np.triu(a["c2"]))
        self.nchan = self.ns * a["n_rad"]
        self.c3 = None
        if a["order"] >= 3:
            L1, nc = a["lmax"] + 1, self.nchan
            K = nc * L1
            k = torch.arange(K, device=DEV)
            use = (k[:, None, None] <= k[None, :, None]) & (k[None, :, None] <= k[None, None, :])
            self.c3 = (t(a["c3"]) * use).reshape(self.ns, nc, L1, nc, L1, nc, L1)
            self.G = _gaunt(a["lmax"], DEV)
        self.v2, self.v3 = t(u["c2"]), t(u["c3"])

    def site(self, z, A):
        """Site energies of centres of species z from A (atoms, channels, lm)."""
        e = self.c0[z] + A[:, :, 0] @ self.c1[z]
        if self.a["order"] >= 2:
            for l in range(self.a["lmax"] + 1):
                B = A[:, :, l * l:(l + 1) ** 2]
                e = e + ((self.c2[z, l] @ B) * B).sum((1, 2))
        if self.c3 is not None:
            n, nc = len(A), self.nchan
            for l1, l2, l3 in _triples(self.a["lmax"]):
                W = self.c3[z, :, l1, :, l2, :, l3].reshape(nc * nc, nc)
                B1, B2, B3 = (A[:, :, l * l:(l + 1) ** 2] for l in (l1, l2, l3))
                g = _block(self.G, l1, l2, l3)
                X = (B1 @ g.reshape(2 * l1 + 1, -1)).reshape(n, nc, 2 * l2 + 1, 2 * l3 + 1)
                P = torch.matmul(B2[:, None], X).permute(0, 3, 2, 1)  # (n, m3, b, a)
                D = P.transpose(2, 3).reshape(n, 2 * l3 + 1, nc * nc) @ W
                e = e + (D * B3.transpose(1, 2)).sum((1, 2))
        return e

    def expensive(self, n, species, pairs, S, weights=None, chunk=1024):
        """(site energies, forces) on the induced subsystem S."""
        a = self.a
        i, j, d = pairs
        use = S[i] & S[j] & (d.square().sum(1) < a["rcut"] ** 2)
        i, j, d = i[use], j[use], d[use]
        E = torch.zeros(n, device=DEV, dtype=torch.float64)
        F = torch.zeros(n, 3, device=DEV, dtype=torch.float64)
        for z in range(self.ns):
            centres = (S & (species == z)).nonzero().reshape(-1)
            for c in centres.split(chunk):
                row = torch.full((n,), -1, device=DEV, dtype=torch.int64)
                row[c] = torch.arange(len(c), device=DEV)
                at = (row[i] >= 0).nonzero().reshape(-1)
                ii, jj = i[at], j[at]
                dd = d[at].requires_grad_(True)
                r = dd.norm(dim=1)
                x, s = 2 * r / a["rcut"] - 1, (1 - (r / a["rcut"]) ** 2) ** 2
                T = [torch.ones_like(x), x]
                for _ in range(2, a["n_rad"]):
                    T.append(2 * x * T[-1] - T[-2])
                R = torch.stack(T[:a["n_rad"]], 1) * s[:, None]
                RY = R[:, :, None] * _ylm(a["lmax"], dd / r[:, None])[:, None, :]
                A = torch.zeros(len(c) * self.ns, *RY.shape[1:], device=DEV, dtype=torch.float64)
                A = A.index_add(0, row[ii] * self.ns + species[jj].long(), RY)
                e = self.site(z, A.reshape(len(c), self.nchan, -1))
                (g,) = torch.autograd.grad(e, dd, torch.ones_like(e) if weights is None else weights[c])
                E[c] = e.detach()
                F.index_add_(0, ii, g).index_add_(0, jj, -g)
        return E, F

    def spline(self, knots, top, x):
        """Clamped uniform cubic B-splines at x (Cox-de Boor)."""
        t = [top * min(max(k - 3, 0), knots - 1) / (knots - 1) for k in range(knots + 6)]
        N = [((x >= t[k]) & (x < t[k + 1])).to(x.dtype) for k in range(len(t) - 1)]
        for q in (1, 2, 3):
            N = [((x - t[k]) / (t[k + q] - t[k]) * N[k] if t[k + q] > t[k] else 0.0)
                 + ((t[k + q + 1] - x) / (t[k + q + 1] - t[k + 1]) * N[k + 1]
                    if t[k + q + 1] > t[k + 1] else 0.0) for k in range(len(N) - 1)]
        return torch.stack([v if torch.is_tensor(v) else torch.zeros_like(x) for v in N], 1)

    def legs(self, i, d):
        """Unordered leg pairs (first, second) with one centre and both legs in
        the 3-body cutoff, as indices of the pairs."""
        at = (d.detach().square().sum(1) < self.u["rcut3"] ** 2).nonzero().reshape(-1)
        c, count = torch.unique_consecutive(i[at], return_counts=True)
        if not len(c):
            return at, at
        most = int(count.max())
        first = torch.cumsum(count, 0) - count
        p, q = torch.triu_indices(most, most, 1, device=DEV)
        on = q[None, :] < count[:, None]
        return at[(first[:, None] + p)[on]], at[(first[:, None] + q)[on]]

    def cheap(self, n, species, pairs, S=None, chunk=4096):
        u = self.u
        i, j, d = pairs
        use = d.square().sum(1) < max(u["rcut2"], u["rcut3"] if u["n_knots3"] else 0.0) ** 2
        if S is not None:
            use &= S[i] & S[j]
        i, j, d = i[use], j[use], d[use]
        E = torch.zeros(n, device=DEV, dtype=torch.float64)
        F = torch.zeros(n, 3, device=DEV, dtype=torch.float64)
        ends = torch.searchsorted(i, torch.arange(0, n + chunk, chunk, device=DEV)).tolist()
        for lo, hi in zip(ends[:-1], ends[1:]):
            if hi == lo:
                continue
            ii, jj, dd = i[lo:hi], j[lo:hi], d[lo:hi].clone().requires_grad_(True)
            r = dd.norm(dim=1)
            B = self.spline(u["n_knots2"], u["rcut2"], r)
            e = torch.zeros(n, device=DEV, dtype=torch.float64)
            e = e.index_add(0, ii, 0.5 * (B * self.v2[species[ii].long(), species[jj].long()]).sum(1))
            if u["n_knots3"]:
                p, q = self.legs(ii, dd)
                side = (dd[q] - dd[p]).norm(dim=1)
                nb = u["n_knots3"] + 2
                leg = self.spline(u["n_knots3"], u["rcut3"], r)
                third = self.spline(u["n_knots3"], 2 * u["rcut3"], side)
                z = species[ii[p]].long()
                for k in range(self.ns):
                    m = z == k if self.ns > 1 else slice(None)
                    V = (leg[p[m]][:, :, None] * leg[q[m]][:, None, :]).reshape(-1, nb * nb)
                    V = ((V @ self.v3[k].reshape(nb * nb, nb)) * third[m]).sum(1)
                    e = e.index_add(0, ii[p[m]], V)
            (g,) = torch.autograd.grad(e.sum(), dd)
            E += e.detach()
            F.index_add_(0, ii, g).index_add_(0, jj, -g)
        return E, F

    def mixed(self, a, x, mode, buffer, masked=False):
        """The force call: what System.compute returns, without flags and counts."""
        n, L, periodic, species = a["n"], a["L"], a["periodic"], a["species"]
        lam = torch.zeros(n, device=DEV, dtype=torch.float64)
        if mode == "expensive":
            lam += 1.0
        elif mode == "mixed":
            for g in a["regions"]:
                c = x[:, g["follow_atom"]] if g.get("follow_atom", -1) >= 0 else torch.tensor(
                    g["center"], device=DEV, dtype=torch.float64)
                d = _fold([x[k] - c[k] for k in range(3)], L, periodic)
                r = torch.sqrt(sum(d[k] ** 2 for k in range(3) if g["type"] == 0 or k != g["axis"]))
                t = (r - g["r_core"]) / g["r_blend"]
                b = 1 - t * t * (3 - 2 * t) if g.get("blend", 0) else 1 - t
                b = torch.where(t < 0, 1.0, torch.where(t < 1, b, 0.0))
                lam = torch.maximum(lam, b)
        reach = max(self.a["rcut"], self.u["rcut2"], buffer)
        pairs = _pairs(x, L, periodic, reach)
        i, j, d = pairs
        close = d.square().sum(1) < buffer * buffer
        S = lam > 0
        near = close & S[j]
        S = S.clone()
        S[i[near]] = True
        E = torch.zeros(n, device=DEV, dtype=torch.float64)
        F = torch.zeros(n, 3, device=DEV, dtype=torch.float64)
        ee, fe = self.expensive(n, species, pairs, S) if mode != "cheap" else (E, F)
        Sc = None
        if masked:
            Sc = lam < 1
            near = close & Sc[j]
            Sc = Sc.clone()
            Sc[i[near]] = True
        ec, fc = self.cheap(n, species, pairs, Sc) if mode != "expensive" else (E, F)
        f = lam[:, None] * fe + (1 - lam[:, None]) * fc
        return dict(forces=f.t().contiguous(), e_exp=ee, e_cheap=ec, lam=lam)


def _exact_md(pot, a, dt, steps, mode, buffer, masked=False):
    ex = _Exact(pot)
    x, v, m = a["pos"].clone(), a["vel"].clone(), a["mass"]
    out = ex.mixed(a, x, mode, buffer, masked)
    energies = []
    for _ in range(steps):
        v = v + 0.5 * dt * KAPPA * out["forces"] / m
        x = _wrap(x + dt * v, a["L"], a["periodic"])
        out = ex.mixed(a, x, mode, buffer, masked)
        v = v + 0.5 * dt * KAPPA * out["forces"] / m
        energies.append(torch.stack([out["e_exp"].sum(), out["e_cheap"].sum(),
                                     (0.5 * m * v.square().sum(0)).sum() / KAPPA]))
    return dict(out, pos=x, vel=v, energies=torch.stack(energies))


def _exact_rows(case, c):
    """Energy and force rows of one configuration by the unknown coefficients."""
    k2, k3 = case["knots2"], case["knots3"]
    _, _, _, (_, rc2), (_, rc3), _ = POTENTIALS["w"]
    ex = object.__new__(_Exact)
    ex.u = dict(n_knots2=k2, rcut2=rc2, n_knots3=k3, rcut3=rc3)
    n = c["n"]
    i, j, d = _pairs(c["pos"], c["L"], [1, 1, 1], rc2)

    def basis(knots, top, r):
        r = r.clone().requires_grad_(True)
        B = ex.spline(knots, top, r)
        dB = torch.stack([torch.autograd.grad(B[:, k].sum(), r, retain_graph=True)[0]
                          for k in range(B.shape[1])], 1)
        return B.detach(), dB

    r = d.norm(dim=1)
    B, dB = basis(k2, rc2, r)
    n2 = k2 - 1
    rows = [0.5 * B[:, :n2].sum(0)]
    f = torch.zeros(3, n, n2, device=DEV, dtype=torch.float64)
    for k in range(3):
        g = 0.5 * dB[:, :n2] * (d[:, k] / r)[:, None]
        f[k].index_add_(0, i, g).index_add_(0, j, -g)
    F = [f]
    if k3:
        nl, nb = k3 - 1, k3 + 2
        p, q = ex.legs(i, d)
        pq = torch.triu_indices(nl, nl, device=DEV)
        e3 = torch.zeros(pq.shape[1] * nb, device=DEV, dtype=torch.float64)
        f3 = torch.zeros(3, n, len(e3), device=DEV, dtype=torch.float64)
        leg, dleg = basis(k3, rc3, r)
        for a, b in zip(p.split(100000), q.split(100000)):
            side = d[b] - d[a]
            rs = side.norm(dim=1)
            T, dT = basis(k3, 2 * rc3, rs)

            def prod(x, y, t):
                v = x[:, pq[0]] * y[:, pq[1]]
                w = x[:, pq[1]] * y[:, pq[0]]
                v = torch.where((pq[0] != pq[1])[None], v + w, v)
                return (v[:, :, None] * t[:, None, :]).reshape(len(x), -1)

            e3 += prod(leg[a], leg[b], T).sum(0)
            ga, gb, gs = (prod(dleg[a], leg[b], T), prod(leg[a], dleg[b], T), prod(leg[a], leg[b], dT))
            for k in range(3):
                va = ga * (d[a, k] / r[a])[:, None] - gs * (side[:, k] / rs)[:, None]
                vb = gb * (d[b, k] / r[b])[:, None] + gs * (side[:, k] / rs)[:, None]
                f3[k].index_add_(0, i[a], va + vb).index_add_(0, j[a], -va).index_add_(0, j[b], -vb)
        rows.append(e3)
        F.append(f3)
    return torch.cat([torch.cat(rows)[None], torch.cat(F, 2).reshape(3 * n, -1)])


def _exact_fit(case, seed):
    soft, hard, y, w, yH, wH = _fit_data(case, seed)
    rows = torch.cat([_exact_rows(case, c) for c in soft])
    AH = torch.cat([_exact_rows(case, c)[:1] for c in hard])
    G, b = rows.t() @ (w[:, None] * rows), rows.t() @ (w * y)
    GH, bH = AH.t() @ (wH[:, None] * AH), AH.t() @ (wH * yH)
    eye = torch.eye(len(b), device=DEV, dtype=torch.float64)

    def solve(lam):
        u = torch.linalg.solve(G + lam * GH + RIDGE * eye, b + lam * bH)
        r = AH @ u - yH
        return lam, u, float((wH * r * r).sum())

    now, low, solves = solve(LAMBDA0), 0.0, 1
    while now[2] > ALPHA and solves <= 24:
        low, now, solves = now[0], solve(10 * now[0]), solves + 1
    high = now
    while low > 0.0 and high[2] <= ALPHA and ALPHA - high[2] >= ALPHA / 10.0:
        now = solve(0.5 * (low + high[0]))
        if now[2] <= ALPHA:
            high = now
        else:
            low = now[0]
    return dict(rows=rows, AH=AH, G=G, b=b, u=high[1], info=dict(lam=high[0], residual=high[2]))


def exact(case, seed):
    kind = case["kind"]
    if kind == "fit":
        return _exact_fit(case, seed)
    if kind == "batch":
        pot = _potential("whe", seed)
        got = [_exact_md(pot, a, 0.2, case["steps"], "mixed", 5.0) for a in _replicas(case, seed)]
        out = {k: torch.cat([g[k] for g in got], -1)
               for k in ("forces", "e_exp", "e_cheap", "lam", "pos", "vel")}
        return dict(out, energies=torch.stack([g["energies"] for g in got], 1))
    n = 2 * case["nx"] * case["ny"] * case["nz"]
    if n * (case["steps"] + 1) > 1500000:
        return None
    a, pot = _atoms(case, seed), _potential(case["potential"], seed)
    buffer = POTENTIALS[case["potential"]][5]
    if kind == "md":
        return _exact_md(pot, a, 1.0, case["steps"], case["mode"], buffer, case["masked"])
    ex = _Exact(pot)
    if kind == "force":
        return ex.mixed(a, a["pos"], case["mode"], buffer, case["masked"])
    m = ex.mixed(a, a["pos"], "cheap" if case["mode"] == "cheap" else case["mode"], buffer)
    pairs = _pairs(a["pos"], a["L"], a["periodic"], max(ex.a["rcut"], buffer))
    S = m["lam"] > 0
    near = (pairs[2].square().sum(1) < buffer * buffer) & S[pairs[1]]
    S = S.clone()
    S[pairs[0][near]] = True
    e, f = ex.expensive(a["n"], a["species"], pairs, S, a["weights"])
    return dict(e=e, grad=-f.t().contiguous())
