"""The engine's kernels at the edges of their tiles, line lengths and atom
groups, against the oracle and exact identities.

Tolerances: H psi FP64 1e-11 and FP32 2e-6 relative (the operator bounds of
the parity tests); a converged FP64 solve 1e-6 Ha per atom and 1e-5 Ha/bohr
(its residual gate, far above rounding); overlaps of FP64 bands 1e-11: sums of
up to 13,000 products of unit vectors, rotated by matrices orthogonal to 1e-14."""
import numpy as np
import pytest

from tests.gpu_helpers import say, half_to_full_index, pack, random_real_function_coeffs
from workloads import configs
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("grid", [
    (10, 9, 75), (96, 10, 9), (9, 120, 12), (125, 9, 10), (16, 128, 9),  # three stages
    (25, 27, 30), (32, 45, 50), (81, 36, 9), (72, 64, 10), (100, 20, 18), (90, 12, 24),
    (9, 9, 9),  # one stage
])
def test_apply_h_line_lengths(grid, prec):
    """Every radix of the in-place LDS lines, odd and even pitches."""
    import paper_1603_02732_amd as sgo
    from oracle.hamiltonian import Setup
    s = workloads.tiny_system("sip", ecut=1.2, grid=grid, nbands=20)
    say("apply_h", grid, prec)
    ctx = sgo.context_from_system(s, sgo.SGO_FP64 if prec == "fp64" else sgo.SGO_FP32)
    st = Setup(s)
    gm, _ = ctx.basis()
    pos, neg = half_to_full_index(gm, st.millers)
    C = random_real_function_coeffs(st.npw, 5, pos, neg, seed=3)
    V = np.random.default_rng(5).standard_normal(st.grid)
    ref = pack(st.apply_h(V, C), pos)
    got = ctx.apply_h(np.transpose(V, (2, 1, 0)), pack(C, pos))
    err = np.abs(got - ref).max() / np.abs(ref).max()
    say("  rel err %.2e" % err)
    assert err < (1e-11 if prec == "fp64" else 2e-6)


@pytest.mark.parametrize("nb", [16, 17, 31, 32, 33, 48, 64, 65, 128, 129, 193])
def test_band_products(nb):
    """Output tiles of the FP64 band products, the overlap's mirrored blocks and
    the subspace kernels' sizes: orthonormal Ritz vectors in ascending order after
    one pass, and their total charge."""
    import paper_1603_02732_amd as sgo
    s = workloads.tiny_system("sip", ecut=4.0, grid=(15, 15, 16), nbands=nb, occupation=configs.FIXED)
    say("bands", nb)
    b = sgo.Batch(1, precision=sgo.SGO_FP64)
    b.add_system(s)
    b.scf(sgo.default_opts(max_iter=1, ncg_first=2, tol_e=1e-10, tol_rho=1e-8))
    st = b.state(0)
    psi = st["psi"]
    dev = np.abs(psi @ psi.T - np.eye(nb)).max()
    say("  |S - 1| %.2e" % dev)
    assert dev < 1e-11
    assert np.all(np.diff(st["eig"]) >= 0)
    assert abs(st["occ"].sum() - 32.0) < 1e-9


@pytest.mark.parametrize("ecut", [12.2, 12.7, 20.0, 31.0])
def test_long_bands(ecut):
    """Bands around one step of 256 threads and of the wide blocks: the FP64
    solve against the FP32 one, whose band kernels hold a band in registers."""
    import paper_1603_02732_amd as sgo
    s = workloads.tiny_system("c", ecut=ecut, grid=(30, 30, 32))
    r = {}
    for prec in (sgo.SGO_FP64, sgo.SGO_FP32):
        ctx = sgo.context_from_system(s, prec)
        ctx.scf(tol_e=1e-7, tol_rho=1e-5, max_iter=150)
        r[prec] = (ctx.energy()[0], ctx.forces())
        n = len(ctx.basis()[0])
    say("ecut %.1f: %d coefficients, dE %.2e, dF %.2e" % (
        ecut, n, r[sgo.SGO_FP64][0] - r[sgo.SGO_FP32][0],
        np.abs(r[sgo.SGO_FP64][1] - r[sgo.SGO_FP32][1]).max()))
    assert abs(r[sgo.SGO_FP64][0] - r[sgo.SGO_FP32][0]) < 1e-5 * 4
    assert np.abs(r[sgo.SGO_FP64][1] - r[sgo.SGO_FP32][1]).max() < 5e-4


def _cluster(symbols, grid):
    lat, pos = configs.cluster_ball(len(symbols), 14.0, 4.5, 2.6, 5)
    return configs.make_system("edge", lat, symbols, pos, 2.2, grid, 2 * len(symbols) + 4, configs.FERMI, "fp64")


@pytest.mark.parametrize("symbols,grid", [
    (["C-G"], (15, 16, 18)),
    (["C-G"] * 7, (16, 15, 15)),
    (["C-G"] * 8, (15, 20, 16)),
    (["C-G"] * 9, (18, 15, 25)),
    (["C-G"] * 3 + ["Si-G"] * 2 + ["C-G"] * 6, (16, 18, 15)),
    (["Si-G"] * 8 + ["C-Gloc"] * 2, (15, 15, 24)),
])
def test_atom_groups_and_grids(symbols, grid):
    """Groups of eight atoms of a species (7, 8, 9, mixed), odd and even grids
    and z remainders of the setup and force kernels, both precisions of the phase
    tables' users: energy, its terms and forces against the dense oracle."""
    import paper_1603_02732_amd as sgo
    from oracle.scf import run_scf
    from oracle.forces import hf_forces
    s = _cluster(symbols, grid)
    ref = run_scf(s)
    F = np.asarray(hf_forces(ref)[0])
    ctx = sgo.context_from_system(s, sgo.SGO_FP64)
    ctx.scf(tol_e=1e-11, tol_rho=1e-9, max_iter=200)
    E, _ = ctx.energy()
    say("atoms", len(symbols), "dE %.2e dF %.2e" % (E - ref["energy"], np.abs(ctx.forces() - F).max()))
    assert abs(E - ref["energy"]) < 1e-6 * len(symbols)
    assert np.abs(ctx.forces() - F).max() < 1e-5


def test_batch_results_match_single_solves():
    """Positions in and results out of a batch in one copy each: moved atoms,
    candidates of different sizes, a second batch of another size, against
    converged solves of one structure (1e-7 Ha, 1e-5 Ha/bohr: the gate)."""
    import paper_1603_02732_amd as sgo
    rng = np.random.default_rng(2)
    gate = dict(tol_e=1e-11, tol_rho=1e-9, max_iter=200)
    for sizes in ((2, 5, 3), (4,)):
        systems = [_cluster(["C-G"] * n, (15, 16, 18)) for n in sizes]
        b = sgo.Batch(len(systems), precision=sgo.SGO_FP64)
        for x in systems:
            b.add_system(x)
        b.scf(sgo.default_opts(max_iter=2))
        moved = [np.array(x["positions"]) + rng.uniform(-0.1, 0.1, (len(x["positions"]), 3)) for x in systems]
        b.reset()
        for i, p in enumerate(moved):
            b.set_atoms(i, p)
        e, f, _ = b.scf(sgo.default_opts(**gate))
        for i, (x, p) in enumerate(zip(systems, moved)):
            one = sgo.context_from_system(dict(x, positions=p.tolist()), sgo.SGO_FP64)
            one.scf(**gate)
            say("candidate %d of %s: dE %.2e" % (i, sizes, e[i] - one.energy()[0]))
            assert abs(e[i] - one.energy()[0]) < 1e-7
            assert np.abs(f[i] - one.forces()).max() < 1e-5


@pytest.mark.parametrize("grid,count", [((72, 64, 10), 5), ((64, 72, 12), 4), ((125, 27, 10), 5), ((45, 50, 16), 3)])
def test_grid_transforms_of_planes_and_lines(grid, count):
    """Grid transforms of whole planes (enough planes to fill the chip, here
    `count` copies) against rows and columns (the structure alone): two
    iterations from the same start, so they differ by FP64 rounding (1e-16 of 20
    Ha, of densities and forces of order one) and what two iterations make of
    it: some 20 steps that divide by level spacings of 0.01 to 0.1 Ha, a factor
    of 1e6 at most, and ten more for the forces' sums over G."""
    import paper_1603_02732_amd as sgo
    s = workloads.tiny_system("c", ecut=2.0, grid=grid)
    r = {}
    for n in (1, count):
        b = sgo.Batch(n, precision=sgo.SGO_FP64)
        for _ in range(n):
            b.add_system(s)
        e, f, _ = b.scf(sgo.default_opts(max_iter=2, tol_e=1e-12, tol_rho=1e-12))
        r[n] = (e[0], f[0], b.state(0)["rho"])
    say("grid", grid, "dE %.2e dF %.2e" % (r[1][0] - r[count][0], np.abs(r[1][1] - r[count][1]).max()))
    assert abs(r[1][0] - r[count][0]) < 2e-9 and np.abs(r[1][1] - r[count][1]).max() < 1e-9
    assert np.abs(r[1][2] - r[count][2]).max() < 1e-10


@pytest.mark.parametrize("nb", [16, 17, 31, 32, 33, 48, 64, 65, 128, 129, 193, 199])
def test_bands_are_ritz_vectors(nb):
    """The bands of one pass are the Ritz vectors of their own span: psi H psi^T
    with H applied anew, in the potential that they were solved in, is diagonal
    and holds their eigenvalues (a wrong H product, congruence, rotation or
    order shows here; orthonormality alone would not).  The occupations add up
    under Fermi filling.  H psi is within 1e-11 of its largest element (the
    operator's bound), below 10 Ha for |k| <= 4 Ha and this potential: 1e-10."""
    import paper_1603_02732_amd as sgo
    s = workloads.tiny_system("sip", ecut=4.0, grid=(15, 15, 16), nbands=nb,
                              occupation=configs.FIXED if nb == 16 else configs.FERMI)
    b = sgo.Batch(1, precision=sgo.SGO_FP64)
    b.add_system(s)
    b.scf(sgo.default_opts(max_iter=1, ncg_first=2, tol_e=1e-10, tol_rho=1e-8))
    st = b.state(0)
    psi = st["psi"]
    ctx = sgo.context_from_system(s, sgo.SGO_FP64)
    H = psi @ ctx.apply_h(st["veff"], psi).T
    dev = np.abs(H - np.diag(st["eig"])).max()
    say("bands %d: |psi H psi^T - eig| %.2e, charge %.12f" % (nb, dev, st["occ"].sum()))
    assert dev < 1e-10
    assert np.abs(psi @ psi.T - np.eye(nb)).max() < 1e-11
    assert np.all(np.diff(st["eig"]) >= 0)
    assert abs(st["occ"].sum() - 32.0) < 1e-9


@pytest.mark.parametrize("graph", [0, 2])
def test_uneven_bands_with_rounds_over_the_gpu(graph):
    """Candidates of 20 to 200 bands in one batch: the Jacobi rounds of the largest
    run over the GPU, and the smaller ones' sweeps end before theirs.  Converged
    energies and forces against solves of one structure (1e-7 Ha, 1e-5 Ha/bohr:
    the gate)."""
    import paper_1603_02732_amd as sgo
    gate = dict(tol_e=1e-10, tol_rho=1e-8, max_iter=100)
    systems = [workloads.tiny_system("sip", ecut=4.0, grid=(15, 15, 16), nbands=nb, seed=11 + k)
               for k, nb in enumerate((40, 200, 20, 65))]
    b = sgo.Batch(len(systems), precision=sgo.SGO_FP64)
    for x in systems:
        b.add_system(x)
    e, f, st = b.scf(sgo.default_opts(use_graph=graph, **gate))
    for i, x in enumerate(systems):
        one = sgo.context_from_system(x, sgo.SGO_FP64)
        one.scf(**gate)
        say("%d bands: dE %.2e dF %.2e" % (x["nbands"], e[i] - one.energy()[0], np.abs(f[i] - one.forces()).max()))
        assert abs(e[i] - one.energy()[0]) < 1e-7
        assert np.abs(f[i] - one.forces()).max() < 1e-5
