"""Timed work of the plane-wave Kohn-Sham engine, through its public entry points.

A structure search evaluates energies and forces of many candidate
structures: single crystals and sheets, populations of clusters solved
together, uneven populations, relaxations and k-point sampled crystals.  `listed()` holds one case of each; `draw` gives more
of the same ranges.  `prepare` builds the handle that a user's program keeps,
`run` is one pass through it (a cold evaluation: `reset` drops the wavefunctions
of the pass before), `work` what the pass cannot do without and `exact` the
converged result of the same discrete functional from plain 64-bit numpy and
torch, where a dense diagonalisation is quick enough.

Results of the forms that do their bulk arithmetic in FP32 are returned as
float32, the precision they carry.
"""
import math

import numpy as np
import torch

import paper_1603_02732_amd as sgo

# Analytic species parameters of the repository's workloads.
SPECIES = {
    "Si-AH": {"Z": 4.0, "local": {"kind": "ah", "alpha": 0.6102, "v1": 3.042, "v2": -1.372},
              "kb": [], "rho0_width": 0.9052},
    "Si-G": {"Z": 4.0, "local": {"kind": "gauss", "rloc": 0.44, "c1": -7.34, "c2": 0.0},
             "kb": [{"l": 0, "r": 0.423, "h": 5.91}, {"l": 1, "r": 0.484, "h": 2.73}],
             "rho0_width": 0.44},
    "C-G": {"Z": 4.0, "local": {"kind": "gauss", "rloc": 0.338, "c1": -8.80, "c2": 1.34},
            "kb": [{"l": 0, "r": 0.303, "h": 9.62}], "rho0_width": 0.338},
    "C-Gloc": {"Z": 4.0, "local": {"kind": "gauss", "rloc": 0.338, "c1": -8.80, "c2": 1.34},
               "kb": [], "rho0_width": 0.338},
}
PRECISION = {"fp64": sgo.SGO_FP64, "fp32": sgo.SGO_FP32, "bf16proj": sgo.SGO_FP32_BF16PROJ}
FERMI = {"kind": "fermi", "sigma": 0.01}
FIXED = {"kind": "fixed"}

# Solver settings.  Crystals are solved to self-consistency in FP64.  The
# others run the unit that a search repeats thousands of times, one pass of
# the self-consistency loop: potential, a few all-band conjugate-gradient
# steps, density, energy and forces (a whole FP32 solve ends where its gate
# happens to be met, at forces that the last bit of its arithmetic moves by
# 1e-3).
SOLVED = dict(tol_e=1e-7, tol_rho=1e-5, max_iter=150)
ONE_PASS = dict(tol_e=1e-5, tol_rho=1.5e-4, max_iter=1, mix_alpha=0.3, kerker_q0=0.3)


def listed():
    return [
        # the subspace step of a small cluster, in a loop that may not allocate
        {"name": "subspace_32", "kind": "subspace", "n": 32, "mode": 3},
        # the same for the largest candidate of an uneven population
        {"name": "subspace_112", "kind": "subspace", "n": 112, "mode": 3},
        # the 8-atom silicon crystal in double precision, solved: energy, forces, stress
        {"name": "crystal_fp64", "kind": "crystal", "species": "Si-AH", "ecut": 8.0, "n1": 24,
         "n2": 24, "n3": 24, "nbands": 20, "filling": "fixed", "gradient": False},
        # a differentiable evaluation, forward and backward: energy, then its
        # gradient in the positions and in the cell (forces and stress)
        {"name": "gradient_fp64", "kind": "crystal", "species": "Si-G", "ecut": 5.0, "n1": 18,
         "n2": 18, "n3": 20, "nbands": 20, "filling": "fermi", "gradient": True},
        # a rough k-point mesh of the 8-atom crystal, s and p projectors
        {"name": "kpoints_fp64", "kind": "kpoints", "species": "Si-G", "ecut": 4.0, "n1": 15,
         "n2": 15, "n3": 15, "nbands": 20, "mesh": "2x2x1"},
        # a conjugate-gradient relaxation step of a few clusters in double precision: three
        # evaluations, two of them warm
        {"name": "relax_4_fp64", "kind": "clusters", "count": 4, "atoms": 9, "box": 20.0,
         "n1": 40, "nbands": 24, "ecut": 10.0, "form": "fp64", "batches": 1, "steps": 1,
         "ncg": 4},
        # one pass of a 24-atom carbon sheet, single structure
        {"name": "sheet_fp32", "kind": "sheet", "atoms": 24, "n1": 48, "n2": 40, "n3": 48,
         "nbands": 56, "ecut": 15.0, "form": "fp32", "ncg": 2},
        # one pass of a search's population of 13-atom clusters, all in one batch
        {"name": "clusters_32", "kind": "clusters", "count": 32, "atoms": 13, "box": 24.0,
         "n1": 48, "nbands": 32, "ecut": 10.0, "form": "fp32", "batches": 1, "steps": 0,
         "ncg": 4},
        # the same population as four batches solved at once on their own streams
        {"name": "clusters_32_split", "kind": "clusters", "count": 32, "atoms": 13, "box": 24.0,
         "n1": 48, "nbands": 32, "ecut": 10.0, "form": "fp32", "batches": 4, "steps": 0,
         "ncg": 4},
        # a few clusters with the projector products on BF16 matrix instructions
        {"name": "clusters_5_bf16proj", "kind": "clusters", "count": 5, "atoms": 13, "box": 24.0,
         "n1": 48, "nbands": 32, "ecut": 10.0, "form": "bf16proj", "batches": 1, "steps": 0,
         "ncg": 4},
        # one pass of an uneven population: 8 to 40 atoms in 12 to 22 bohr cells
        {"name": "uneven_24", "kind": "uneven", "count": 24, "atoms_max": 40, "ecut": 15.0,
         "form": "fp32", "ncg": 1},
        # one pass of a large sheet: long grid lines, more than 160 bands
        {"name": "large_sheet", "kind": "sheet", "atoms": 72, "n1": 80, "n2": 50, "n3": 40,
         "nbands": 164, "ecut": 15.0, "form": "fp32", "ncg": 1},
    ]


def _smooth(n):
    """Smallest FFT length 2^a 3^b 5^c >= n."""
    while True:
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1:
            return n
        n += 1


def _holds(length, ecut):
    """Smallest FFT length whose grid holds the wavefunction sphere."""
    return 2 * int(math.sqrt(2 * ecut) * length / (2 * math.pi)) + 1


def draw(rng):
    kind = rng.choice(["subspace", "crystal", "kpoints", "sheet", "clusters", "clusters",
                       "uneven"])
    if kind == "subspace":
        return {"kind": kind, "n": int(round(math.exp(rng.uniform(math.log(6), math.log(256))))),
                "mode": rng.choice([1, 3, 3])}
    if kind == "crystal":
        ecut = round(rng.uniform(3.0, 8.0), 2)
        n = [_smooth(_holds(10.26, ecut) + rng.randint(0, 6)) for _ in range(3)]
        species = rng.choice(["Si-AH", "Si-G"])
        return {"kind": kind, "species": species, "ecut": ecut, "n1": n[0], "n2": n[1],
                "n3": n[2], "nbands": rng.randint(19, 28),
                "filling": "fixed" if species == "Si-AH" else "fermi",
                "gradient": rng.random() < 0.5}
    if kind == "kpoints":
        ecut = round(rng.uniform(2.5, 4.5), 2)
        n = [_smooth(_holds(10.26, ecut) + 2 + rng.randint(0, 3)) for _ in range(3)]
        return {"kind": kind, "species": rng.choice(["Si-AH", "Si-G"]), "ecut": ecut, "n1": n[0],
                "n2": n[1], "n3": n[2], "nbands": rng.randint(18, 22),
                "mesh": rng.choice(["2x1x1", "2x2x1", "1x1x2"])}
    form = rng.choice(["fp32", "fp32", "bf16proj"])
    if kind == "sheet":
        atoms = 2 * rng.randint(4, 36)
        ecut = round(rng.uniform(8.0, 15.0), 2)
        n = [_smooth(max(_holds(a, ecut), math.ceil(a / 0.375))) for a in _sheet_lengths(atoms)]
        return {"kind": kind, "atoms": atoms, "n1": n[0], "n2": n[1], "n3": n[2],
                "nbands": 2 * atoms + 2 * rng.randint(3, 10), "ecut": ecut, "form": form,
                "ncg": rng.randint(1, 2) if atoms <= 24 else 1}
    if kind == "clusters":
        atoms = rng.randint(3, 13)
        box = round(rng.uniform(18.0, 24.0), 2)
        ecut = round(rng.uniform(7.0, 10.0), 2)
        case = {"kind": kind, "atoms": atoms, "box": box,
                "n1": _smooth(max(_holds(box, ecut), math.ceil(box / 0.5))),
                "nbands": 2 * atoms + 2 * rng.randint(2, 4), "ecut": ecut}
        if rng.random() < 0.3:
            return dict(case, form="fp64", count=rng.randint(1, 8), batches=1, ncg=4,
                        steps=rng.randint(0, 1))
        count = int(round(math.exp(rng.uniform(0, math.log(32)))))
        return dict(case, form=form, count=count, steps=0, ncg=rng.randint(2, 4),
                    batches=1 if count < 8 else rng.choice([1, 2, 4]))
    return {"kind": kind, "count": rng.randint(2, 24), "atoms_max": rng.randint(12, 40),
            "ecut": round(rng.uniform(9.0, 15.0), 2), "form": form, "ncg": 1}


# ------------------------------------------------------------------ inputs

def _system(lattice, species, positions, ecut, grid, nbands, occupation):
    return {"lattice": np.asarray(lattice, dtype=float).tolist(),
            "species": {species: SPECIES[species]}, "symbols": [species] * len(positions),
            "positions": np.asarray(positions, dtype=float).tolist(), "ecut": ecut,
            "grid": [int(n) for n in grid], "nbands": int(nbands), "occupation": occupation}


_DIAMOND = np.array([(0, 0, 0), (0, 2, 2), (2, 0, 2), (2, 2, 0), (1, 1, 1), (1, 3, 3), (3, 1, 3),
                     (3, 3, 1)]) / 4.0


def _diamond(case, rng, occupation):
    """Silicon's cubic cell, every coordinate moved a little."""
    pos = 10.26 * _DIAMOND + rng.uniform(-0.1, 0.1, size=(8, 3))
    return _system(10.26 * np.eye(3), case["species"], pos, case["ecut"],
                   (case["n1"], case["n2"], case["n3"]), case["nbands"], occupation)


def _sheet_rows(atoms):
    """Rows of a sheet, as near square as its atom count allows."""
    return max(r for r in range(1, int(math.sqrt(atoms)) + 1) if atoms % r == 0)


def _sheet_lengths(atoms):
    """Cell of a sheet: the 24-atom workload's areal density at every size."""
    rows = _sheet_rows(atoms)
    return round(14.0 / 6 * atoms / rows, 3), round(12.1 / 4 * rows, 3), 15.0


def _sheet(case, rng):
    """A flat carbon sheet: staggered rows at the workload's areal density."""
    n = case["atoms"]
    lx, ly, lz = _sheet_lengths(n)
    rows = _sheet_rows(n)
    cols = n // rows
    pos = [[(c + 0.5 * (r % 2) + 0.25) * lx / cols, (r + 0.5) * ly / rows, 0.5 * lz]
           for r in range(rows) for c in range(cols)]
    pos = np.array(pos)
    pos[:, :2] += rng.uniform(-0.12, 0.12, size=(n, 2))
    return _system(np.diag([lx, ly, lz]), "C-Gloc", pos, case["ecut"],
                   (case["n1"], case["n2"], case["n3"]), case["nbands"], FERMI)


def _placed(rng, n, lengths, sample, dmin, periodic):
    """n random positions at least dmin apart."""
    while True:
        pos, fails = np.zeros((0, 3)), 0
        while len(pos) < n and fails < 2000:
            p = sample()
            d = pos - p
            if periodic:
                d -= np.round(d / lengths) * lengths
            if len(pos) == 0 or (d * d).sum(1).min() >= dmin * dmin:
                pos = np.vstack([pos, p])
            else:
                fails += 1
        if len(pos) == n:
            return pos


def _clusters(case, rng):
    box = np.full(3, case["box"])

    def sample():
        while True:
            p = rng.uniform(-5.0, 5.0, size=3)
            if (p * p).sum() <= 25.0:
                return 0.5 * box + p

    grid = (case["n1"],) * 3
    return [_system(np.diag(box), "C-G", _placed(rng, case["atoms"], box, sample, 3.5, False),
                    case["ecut"], grid, case["nbands"], FERMI) for _ in range(case["count"])]


def _uneven(case, rng):
    out = []
    # the atom counts and cells are the case's, the positions the seed's
    shape = np.random.default_rng([case["count"], case["atoms_max"]])
    for _ in range(case["count"]):
        n = int(shape.integers(8, case["atoms_max"] + 1))
        lengths = (np.full(3, shape.uniform(12.0, 22.0)) if shape.uniform() < 0.5
                   else shape.uniform(12.0, 22.0, size=3))
        pos = _placed(rng, n, lengths, lambda: rng.uniform(0, 1, size=3) * lengths, 2.4, True)
        grid = [_smooth(math.ceil(a / 0.375)) for a in lengths]
        nb = math.ceil(1.4 * 2 * n)
        out.append(_system(np.diag(lengths), "C-G", pos, case["ecut"], grid, nb + nb % 2, FERMI))
    return out


def _systems(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "crystal":
        return [_diamond(case, rng, FIXED if case["filling"] == "fixed" else FERMI)]
    if kind == "kpoints":
        return [_diamond(case, rng, FERMI)]
    if kind == "sheet":
        return [_sheet(case, rng)]
    return _clusters(case, rng) if kind == "clusters" else _uneven(case, rng)


def _mesh(text):
    """Monkhorst-Pack mesh reduced by time reversal: fractional k, weights."""
    q = [int(n) for n in text.split("x")]
    ks = {}
    for i in range(q[0]):
        for j in range(q[1]):
            for k in range(q[2]):
                f = tuple(round((2 * r + 1 - n) / (2.0 * n), 9) for r, n in zip((i, j, k), q))
                m = tuple(-x + 0.0 for x in f)
                key = max(f, m)
                ks[key] = ks.get(key, 0.0) + 1.0 / (q[0] * q[1] * q[2])
    return np.array(list(ks)), np.array(list(ks.values()))


def _subspace_matrices(n, seed):
    """Overlap and Hamiltonian of bands after a line minimisation: nearly
    orthonormal and nearly diagonal, with the levels of a valence band."""
    g = np.random.default_rng(seed)
    a, b = g.normal(size=(2, n, n)) / math.sqrt(n)
    levels = np.sort(g.uniform(-0.9, 0.6, size=n))
    S = np.eye(n) + 0.05 * (a + a.T)
    H = np.diag(levels) + 0.05 * (b + b.T)
    return S, H


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    if case["kind"] == "subspace":
        n = case["n"]
        S, H = _subspace_matrices(n, seed)
        s.S = torch.from_numpy(S).cuda()
        s.H = torch.from_numpy(H).cuda()
        s.M = torch.zeros(n, n, dtype=torch.float64, device="cuda")
        s.eps = torch.zeros(n, dtype=torch.float64, device="cuda")
        s.status = torch.zeros(1, dtype=torch.int32, device="cuda")
        return s
    systems = _systems(case, seed)
    if case["kind"] in ("clusters", "uneven"):
        nb = case.get("batches", 1)
        s.batches, s.streams = [], []
        per = -(-len(systems) // nb)
        for k in range(0, len(systems), per):
            part = systems[k:k + per]
            batch = sgo.Batch(len(part), precision=PRECISION[case["form"]])
            for x in part:
                batch.add_system(x)
            if nb > 1:
                s.streams.append(torch.cuda.Stream())
                batch.set_stream(s.streams[-1].cuda_stream)
            s.batches.append(batch)
        s.positions = [np.array(x["positions"]) for x in systems]
    else:
        s.ctx = sgo.context_from_system(systems[0], PRECISION[case.get("form", "fp64")])
        if case["kind"] == "kpoints":
            s.ctx.set_kpoints(*_mesh(case["mesh"]))
        s.positions = torch.tensor(systems[0]["positions"], dtype=torch.float64)
        s.lattice = torch.tensor(systems[0]["lattice"], dtype=torch.float64)
    if "ncg" in case:
        s.opts = sgo.default_opts(ncg_first=case["ncg"], **ONE_PASS)
    else:
        s.opts = sgo.default_opts(**SOLVED)
    return s


# -------------------------------------------------------------------- pass

def _typed(case, out):
    """Results in the precision that the form carries."""
    if case.get("form", "fp64") == "fp64":
        return out
    return {k: np.asarray(v, dtype=np.float32) for k, v in out.items()}


def run(s):
    case = s.case
    if case["kind"] == "subspace":
        sgo.subspace_solve_noalloc(s.S.data_ptr(), s.H.data_ptr() if case["mode"] == 3 else None,
                                   s.M.data_ptr(), s.eps.data_ptr(), case["n"], case["mode"],
                                   status=s.status.data_ptr(),
                                   stream=torch.cuda.current_stream().cuda_stream)
        if case["mode"] == 1:
            return {"M": s.M, "status": s.status}
        return {"M": s.M, "eps": s.eps, "status": s.status}
    if case["kind"] in ("clusters", "uneven"):
        for b in s.batches:
            b.reset()
        if case.get("steps", 0):
            for i, p in enumerate(s.positions):
                s.batches[0].set_atoms(i, p)
            e, f, x, _ = s.batches[0].relax_cg(case["steps"], opts=s.opts)
            return _typed(case, {"energies": e, "forces": np.concatenate(f),
                                 "positions": np.concatenate(x)})
        if len(s.batches) == 1:
            e, f, _ = s.batches[0].scf(s.opts)
        else:
            e, f, _ = sgo.batches_scf(s.batches, s.opts)
        return _typed(case, {"energies": e, "forces": np.concatenate(f)})
    s.ctx.reset()
    if case.get("gradient"):
        from paper_1603_02732_amd.autograd import scf_energy
        pos = s.positions.clone().requires_grad_(True)
        lat = s.lattice.clone().requires_grad_(True)
        e = scf_energy(pos, s.ctx, s.opts, lat)
        e.backward()
        return {"energy": e.detach(), "positions": pos.grad, "lattice": lat.grad}
    s.ctx.scf(s.opts, allow_notconv=True)
    e, _ = s.ctx.energy()
    out = {"energy": np.array([e]), "forces": s.ctx.forces()}
    out["density"], out["potential"] = s.ctx.density()
    if case["kind"] == "kpoints":
        out["levels"], out["occupations"] = s.ctx.kpoint_eigenvalues()
    else:
        out["stress"] = s.ctx.stress()
    return _typed(case, out)


# ------------------------------------------------------------ needed work

def work(case):
    """Bytes: inputs read and results written once, bands and density once per
    self-consistency iteration.  Operations: per application of H the line
    transforms of the sphere's columns and of the planes, and the band products
    of one subspace step, at the applications that the pass makes."""
    if case["kind"] == "subspace":
        n = case["n"]
        diag = case["mode"] == 3
        return {"bytes": 8 * (3 if diag else 2) * n * n, "flops": (9 if diag else 2 / 3) * n ** 3}
    form = case.get("form", "fp64")
    real = 8 if form == "fp64" else 4
    # applications of H: one pass, or a solve's fifteen or so
    applications = 1 + case["ncg"] if "ncg" in case else 15 * 4
    densities = 1 if "ncg" in case else 15
    complex_bands = 1
    if case["kind"] == "uneven":
        sizes = [(17.0 ** 3, (17.0 / 0.375) ** 3, 1.4 * (8 + case["atoms_max"]))] * case["count"]
    elif case["kind"] == "clusters":
        sizes = [(case["box"] ** 3, case["n1"] ** 3, case["nbands"])] * case["count"]
        applications *= 1 + 2 * case["steps"]
        densities *= 1 + 2 * case["steps"]
    else:
        volume = 10.26 ** 3
        if case["kind"] == "sheet":
            volume = math.prod(_sheet_lengths(case["atoms"]))
        if case["kind"] == "kpoints":  # complex bands: no pairing of two in one transform
            complex_bands = 2 * len(_mesh(case["mesh"])[0])
        sizes = [(volume, case["n1"] * case["n2"] * case["n3"], case["nbands"])]
    total = {"bytes": 0.0, "flops": 0.0}
    for volume, ntot, nb in sizes:
        k = (2 * case["ecut"]) ** 1.5 * volume / (6 * math.pi ** 2)  # real coefficients of a band
        transform = 0.5 * 5 * ntot * math.log2(ntot) * nb / 2  # half the columns are empty
        total["flops"] += complex_bands * (applications * (2 * transform + 8 * k * nb * nb)
                                           + densities * transform)
        total["bytes"] += (complex_bands * 2 * applications * k * nb * real
                           + densities * 3 * 8 * ntot)
    return total


# --------------------------------------------------------- 64-bit reference

def _pz81(rho):
    """Perdew-Zunger exchange-correlation energy per electron and potential."""
    r = np.maximum(rho, 1e-30)
    rs = (3 / (4 * np.pi * r)) ** (1 / 3)
    ex = -0.75 * (3 / np.pi) ** (1 / 3) * r ** (1 / 3)
    q = np.sqrt(rs)
    den = 1 + 1.0529 * q + 0.3334 * rs
    far = -0.1423 / den
    vfar = far * (1 + 7 / 6 * 1.0529 * q + 4 / 3 * 0.3334 * rs) / den
    ln = np.log(rs)
    near = 0.0311 * ln - 0.048 + 0.0020 * rs * ln - 0.0116 * rs
    vnear = 0.0311 * ln - 0.048 - 0.0311 / 3 + 2 / 3 * 0.0020 * rs * ln + (2 * -0.0116 - 0.0020) / 3 * rs
    low = rs >= 1
    dead = rho <= 1e-30
    return (np.where(dead, 0, ex + np.where(low, far, near)),
            np.where(dead, 0, 4 / 3 * ex + np.where(low, vfar, vnear)))


def _local(sp, g2):
    """Transform of the local potential at |G|^2 > 0, and its finite part at 0."""
    p, Z = sp["local"], sp["Z"]
    if p["kind"] == "ah":
        a = p["alpha"]
        e = np.exp(-g2 / (4 * a))
        short = (np.pi / a) ** 1.5 * e * (p["v1"] + p["v2"] * (1.5 / a - g2 / (4 * a * a)))
        zero = np.pi * Z / a + (np.pi / a) ** 1.5 * (p["v1"] + 1.5 * p["v2"] / a)
    else:
        r2 = p["rloc"] ** 2
        e = np.exp(-0.5 * g2 * r2)
        pre = (2 * np.pi * r2) ** 1.5
        short = pre * e * (p["c1"] + p["c2"] * (3 - g2 * r2))
        zero = 2 * np.pi * Z * r2 + pre * (p["c1"] + 3 * p["c2"])
    return -4 * np.pi * Z / g2 * e + short, zero


def _projectors(system, q, omega):
    """Columns beta(q), strengths and owners; one column per (atom, l, m)."""
    q2 = (q * q).sum(1)
    cols, h, owner = [], [], []
    for i, (name, pos) in enumerate(zip(system["symbols"], np.array(system["positions"]))):
        phase = np.exp(-1j * (q @ pos)) / math.sqrt(omega)
        for ch in system["species"][name]["kb"]:
            r, l = ch["r"], ch["l"]
            radial = (4 * np.pi ** 1.5 * r ** (l + 1.5) * np.exp(-0.5 * q2 * r * r)
                      / math.sqrt(math.gamma(l + 1.5)))
            ang = [math.sqrt(1 / (4 * np.pi)) * np.ones(len(q))] if l == 0 else \
                [-1j * math.sqrt(3 / (4 * np.pi)) * q[:, a] for a in range(3)]
            for y in ang:
                cols.append(radial * y * phase)
                h.append(ch["h"])
                owner.append(i)
    cols = np.array(cols).T if cols else np.zeros((len(q), 0), dtype=complex)
    return cols, np.array(h), np.array(owner, dtype=int)


def _ewald(lattice, Z, R):
    """Energy and forces of the ions in a neutralising background."""
    omega = abs(np.linalg.det(lattice))
    B = 2 * np.pi * np.linalg.inv(lattice).T
    eta = math.sqrt(np.pi) * (len(Z) / omega ** 2) ** (1 / 6)

    def ball(rows, radius):
        inv = np.linalg.inv(rows)
        m = [int(radius * np.linalg.norm(inv[:, i])) + 1 for i in range(3)]
        idx = np.stack(np.meshgrid(*[np.arange(-k, k + 1) for k in m], indexing="ij"), -1)
        return idx.reshape(-1, 3) @ rows

    L = ball(lattice, 6.2 / eta + np.linalg.norm(lattice.sum(0)))
    E, F = 0.0, np.zeros((len(Z), 3))
    for i in range(len(Z)):
        d = (R[i] - R)[:, None, :] + L[None]
        r = np.sqrt((d * d).sum(-1))
        use = (r > 1e-9) & (r < 6.5 / eta)
        r = np.where(use, r, 1.0)
        ec = torch.special.erfc(torch.from_numpy(eta * r)).numpy()
        E += 0.5 * Z[i] * (Z[:, None] * np.where(use, ec / r, 0)).sum()
        w = (ec / r + 2 * eta / math.sqrt(np.pi) * np.exp(-(eta * r) ** 2)) / (r * r)
        F[i] += Z[i] * ((Z[:, None] * np.where(use, w, 0))[..., None] * d).sum((0, 1))
    G = ball(B, 12.4 * eta)
    g2 = (G * G).sum(1)
    G, g2 = G[g2 > 1e-12], g2[g2 > 1e-12]
    ph = np.exp(1j * (G @ R.T))
    S = ph @ Z
    w = np.exp(-g2 / (4 * eta * eta)) / g2
    E += 2 * np.pi / omega * (w * abs(S) ** 2).sum() - eta / math.sqrt(np.pi) * (Z * Z).sum()
    E -= np.pi * Z.sum() ** 2 / (2 * omega * eta * eta)
    F += 4 * np.pi / omega * Z[:, None] * ((w[:, None] * np.imag(S.conj()[:, None] * ph)).T @ G)
    return E, F


def _levels(st, veff, k, nb):
    """Lowest nb eigenpairs of the dense H of one k-point."""
    vG = np.fft.fftn(veff) / veff.size
    m = st["millers"][k]
    d = m[:, None, :] - m[None, :, :]
    N = veff.shape
    H = vG[d[..., 0] % N[0], d[..., 1] % N[1], d[..., 2] % N[2]]
    beta, h, _ = st["beta"][k]
    H = H + (beta * h) @ beta.conj().T
    H[np.arange(len(m)), np.arange(len(m))] += st["kin"][k]
    if not st["gamma"]:
        w, v = torch.linalg.eigh(torch.from_numpy(H))
        return w.numpy()[:nb], v.numpy()[:, :nb]
    # real bands at Gamma: sums and differences of +-G halve the dense problem
    pos, neg = st["pair"]
    n = len(pos)
    A, Bm = H[np.ix_(pos, pos)], H[np.ix_(pos, neg)]
    s = np.where(pos == neg, math.sqrt(0.5), 1.0)
    cc = (A + Bm).real * s[:, None] * s
    ss = (A - Bm).real
    cs = (-A + Bm).imag * s[:, None]
    R = np.block([[cc, cs[:, 1:]], [cs.T[1:], ss[1:, 1:]]])
    w, v = torch.linalg.eigh(torch.from_numpy(R))
    v = v.numpy()[:, :nb]
    a = v[:n] * s[:, None]
    b = np.vstack([np.zeros((1, nb)), v[n:]])
    C = np.zeros((len(m), nb), dtype=complex)
    C[neg] = (a - 1j * b) / math.sqrt(2)
    C[pos] = np.where((pos == neg)[:, None], a * math.sqrt(2), (a + 1j * b) / math.sqrt(2))
    return w.numpy()[:nb], C


def _fill(eps, wk, nelec, occ):
    """Occupations of [k][band] levels and the entropy term -sigma S."""
    if occ["kind"] == "fixed":
        f = np.zeros_like(eps)
        f[:, :int(round(nelec / 2))] = 2.0
        return f, 0.0
    sg = occ["sigma"]
    lo, hi = eps.min() - 40 * sg, eps.max() + 40 * sg
    for _ in range(200):
        mu = 0.5 * (lo + hi)
        g = 1 / (1 + np.exp(np.clip((eps - mu) / sg, -500, 500)))
        if (wk[:, None] * 2 * g).sum() > nelec:
            hi = mu
        else:
            lo = mu
    a, b = np.clip(g, 1e-300, 1), np.clip(1 - g, 1e-300, 1)
    return 2 * g, 2 * sg * (wk[:, None] * (a * np.log(a) + b * np.log(b))).sum()


def _reference(system, kfrac, wk):
    """Self-consistent energy, forces, levels and occupations by dense
    diagonalisation."""
    A = np.array(system["lattice"])
    R = np.array(system["positions"])
    omega = abs(np.linalg.det(A))
    B = 2 * np.pi * np.linalg.inv(A).T
    N = system["grid"]
    ntot = N[0] * N[1] * N[2]
    Z = np.array([system["species"][x]["Z"] for x in system["symbols"]])
    nb, occ = system["nbands"], system["occupation"]
    freq = [np.rint(np.fft.fftfreq(n) * n).astype(int) for n in N]
    mg = np.stack(np.meshgrid(*freq, indexing="ij"), -1)
    G = mg @ B
    g2 = (G * G).sum(-1)
    inside = np.all(2 * np.abs(mg) < np.array(N), axis=-1)
    nz = inside & (g2 > 1e-12)
    safe = np.where(g2 > 1e-12, g2, 1.0)
    vloc = np.zeros(N, dtype=complex)
    rho0 = np.zeros(N, dtype=complex)
    tables = {}
    for name, sp in system["species"].items():
        v, v0 = _local(sp, safe)
        tables[name] = np.where(nz, v, np.where(inside, v0, 0))
        at = R[[x == name for x in system["symbols"]]]
        S = np.zeros(N, dtype=complex)
        for r in at:
            S += np.exp(-1j * (G @ r))
        vloc += tables[name] * S / omega
        rho0 += np.where(inside, sp["Z"] * np.exp(-0.5 * g2 * sp["rho0_width"] ** 2) * S / omega, 0)
    e_ion, F = _ewald(A, Z, R)
    st = {"millers": [], "kin": [], "beta": [], "q": [], "gamma": not np.any(kfrac)}
    for k in kfrac:
        box = [int(math.sqrt(2 * system["ecut"]) * np.linalg.norm(a) / (2 * np.pi) + abs(x)) + 1
               for a, x in zip(A, k)]
        m = np.stack(np.meshgrid(*[np.arange(-b, b + 1) for b in box], indexing="ij"), -1).reshape(-1, 3)
        q = (m + k) @ B
        keep = 0.5 * (q * q).sum(1) <= system["ecut"]
        st["millers"].append(m[keep])
        st["q"].append(q[keep])
        st["kin"].append(0.5 * (q[keep] ** 2).sum(1))
        st["beta"].append(_projectors(system, q[keep], omega))
    if st["gamma"]:
        at = {tuple(x): i for i, x in enumerate(st["millers"][0])}
        half = [x for x in at if x > (0, 0, 0)]
        st["pair"] = (np.array([at[0, 0, 0]] + [at[x] for x in half]),
                      np.array([at[0, 0, 0]] + [at[-x[0], -x[1], -x[2]] for x in half]))
    rho = np.fft.ifftn(rho0).real * ntot
    ins, res, last = [], [], None
    for _ in range(60):
        rG = np.fft.fftn(rho) / ntot
        vh = np.fft.ifftn(np.where(nz, 4 * np.pi * rG / safe, 0) + vloc).real * ntot
        veff = vh + _pz81(np.maximum(rho, 0))[1]
        eps, C = zip(*[_levels(st, veff, k, nb) for k in range(len(kfrac))])
        eps = np.array(eps)
        f, ts = _fill(eps, wk, Z.sum(), occ)
        out = np.zeros(N)
        for k, w in enumerate(wk):
            m = st["millers"][k]
            for i in np.nonzero(f[k] > 1e-18)[0]:
                u = np.zeros(N, dtype=complex)
                u[m[:, 0] % N[0], m[:, 1] % N[1], m[:, 2] % N[2]] = C[k][:, i]
                out += w * f[k, i] * np.abs(np.fft.ifftn(u) * ntot) ** 2 / omega
        oG = np.fft.fftn(out) / ntot
        energy = e_ion + ts + omega * (vloc.conj() * oG).real[inside].sum()
        energy += 0.5 * omega * (4 * np.pi * np.abs(oG[nz]) ** 2 / g2[nz]).sum()
        energy += omega / ntot * (np.maximum(out, 0) * _pz81(np.maximum(out, 0))[0]).sum()
        P = [st["beta"][k][0].conj().T @ C[k] for k in range(len(kfrac))]
        for k, w in enumerate(wk):
            energy += w * (f[k] * (st["kin"][k][:, None] * np.abs(C[k]) ** 2).sum(0)).sum()
            energy += w * (f[k] * st["beta"][k][1][:, None] * np.abs(P[k]) ** 2).sum()
        r = out - rho
        if np.abs(r).sum() * omega / ntot / Z.sum() < 1e-10 and last is not None and abs(energy - last) < 1e-11:
            break
        last = energy
        ins, res = (ins + [rho])[-8:], (res + [r])[-8:]
        n = len(ins)
        M = np.ones((n + 1, n + 1))
        M[n, n] = 0
        gram = np.array([[np.vdot(a, b) for b in res] for a in res])
        M[:n, :n] = gram / abs(np.diag(gram)).max()
        c = np.linalg.lstsq(M, np.eye(n + 1)[n], rcond=None)[0][:n]
        step = sum(a * b for a, b in zip(c, res))
        step = np.fft.ifftn(np.where(g2 > 1e-12, g2 / (g2 + 0.64), 0) * np.fft.fftn(step)).real
        rho = sum(a * b for a, b in zip(c, ins)) + 0.5 * step
    for i, name in enumerate(system["symbols"]):
        z = tables[name] * np.exp(1j * (G @ R[i])) * oG
        F[i] += (G[nz] * z.imag[nz][:, None]).sum(0)
    for k, w in enumerate(wk):
        beta, h, owner = st["beta"][k]
        for a in range(3):
            dP = (-1j * st["q"][k][:, a][:, None] * beta).conj().T @ C[k]
            np.add.at(F[:, a], owner, -2 * w * (f[k] * h[:, None] * (P[k].conj() * dP).real).sum(1))
    # the library's grids run [z][y][x], its potential is that of the input density
    return energy, F, eps, f, out.transpose(2, 1, 0)


def exact(case, seed):
    kind = case["kind"]
    if kind == "subspace":
        S, H = _subspace_matrices(case["n"], seed)
        W = np.linalg.inv(np.linalg.cholesky(S))
        if case["mode"] == 1:
            return {"M": W.T, "status": None}
        # eigenvectors have no unique sign: the levels alone are determined
        return {"M": None, "eps": np.linalg.eigvalsh(W @ H @ W.T), "status": None}
    if case.get("form", "fp64") != "fp64" or kind not in ("crystal", "kpoints"):
        return None  # populations, sheets and the large cell: minutes of dense algebra
    system = _systems(case, seed)[0]
    if kind == "kpoints":
        k, w = _mesh(case["mesh"])
    else:
        k, w = np.zeros((1, 3)), np.ones(1)
    e, F, eps, f, rho = _reference(system, k, w)
    if case.get("gradient"):
        # the cell's gradient (stress) has no short dense form here
        return {"energy": torch.tensor(e), "positions": torch.from_numpy(-F), "lattice": None}
    if kind == "kpoints":
        return {"energy": np.array([e]), "forces": F, "density": rho, "potential": None,
                "levels": eps, "occupations": f}
    return {"energy": np.array([e]), "forces": F, "density": rho, "potential": None,
            "stress": None}
