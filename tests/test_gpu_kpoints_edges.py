"""k-point solves at the edges of their kernels' ranges against the oracle's
dense k-point SCF, at two general k-points: band counts around the subspace
kernels' sizes (32 and 64 in LDS, more in global memory; odd and even), grids
whose lines and size select each transform path (lines to 16, 20 and 32 with
the grid in LDS; a grid beyond it), and an element without projectors.
Tolerances as in the k-point oracle test: 1e-6 Ha per atom, 1e-4 Ha/bohr,
eigenvalues of bands that hold charge 1e-5."""
import numpy as np
import pytest

from tests.gpu_helpers import say
import workloads

pytestmark = pytest.mark.gpu
K = [[0.25, 0.1, 0.0], [-0.1, 0.5, 0.3]]
W = [1.0, 3.0]


def _check(s):
    import paper_1603_02732_amd as sgo
    from oracle.kpoints import run_scf_k, hf_forces_k
    ref = run_scf_k(s, K, W)
    Fref, _ = hf_forces_k(ref)
    ctx = sgo.context_from_system(s, sgo.SGO_FP64)
    ctx.set_kpoints(K, W)
    info = ctx.scf(tol_e=1e-10, tol_rho=1e-8, max_iter=200)
    E, _ = ctx.energy()
    eig, occ = ctx.kpoint_eigenvalues()
    nat = len(s["symbols"])
    say("  dE %.2e  max dF %.2e" % (E - ref["energy"], np.abs(ctx.forces() - Fref).max()))
    assert info["converged"]
    assert abs(E - ref["energy"]) < 1e-6 * nat
    assert np.abs(ctx.forces() - Fref).max() < 1e-4
    for ik in range(len(K)):
        f = np.asarray(ref["occupations"][ik])
        held = f > 1e-6
        assert np.abs(eig[ik][held] - np.asarray(ref["eigenvalues"][ik])[held]).max() < 1e-5
        assert np.abs(occ[ik] - f).max() < 1e-5


@pytest.mark.parametrize("nb", [18, 31, 32, 33, 63, 64, 65])
def test_band_counts(nb):
    say("k-point bands %d" % nb)
    _check(workloads.tiny_system("sip", ecut=3.0, grid=(12, 12, 12), nbands=nb))


@pytest.mark.parametrize("grid", [(15, 12, 16), (18, 12, 20), (20, 20, 20), (12, 32, 15), (27, 12, 12), (12, 12, 36),
                                  (24, 24, 20)])
def test_grids(grid):
    say("k-point grid", grid)
    _check(workloads.tiny_system("sip", ecut=3.0, grid=grid))


def test_no_projectors():
    say("k-points, local potential only, fixed occupations")
    _check(workloads.tiny_system("si", ecut=3.0, grid=(12, 12, 12)))


def _solve(s, K, W):
    import paper_1603_02732_amd as sgo
    ctx = sgo.context_from_system(s, sgo.SGO_FP64)
    ctx.set_kpoints(K, W)
    assert ctx.scf(tol_e=1e-10, tol_rho=1e-8, max_iter=200)["converged"]
    return ctx


@pytest.mark.parametrize("grid,copies", [(48, 16), (12, 260)])
def test_many_k_points_in_chunks(grid, copies):
    """More k-points than one chunk of grids (48^3: 14 k-points of 256 MB) or of
    density parts (512 k-points) holds: two k-points, each `copies` times over,
    against the two alone; and the device memory that the chunk allows: 256 MB
    of grids and each k-point's own arrays (10 bands, fewer than 300
    coefficients: under 1 MB), 16 MB for the allocations' granularity."""
    import torch
    s = workloads.tiny_system("c", ecut=3.0, grid=(grid,) * 3)
    _solve(workloads.tiny_system("c", ecut=3.0, grid=(12, 12, 36)), K, W)  # one-time allocations
    free = [torch.cuda.mem_get_info()[0]]
    few = _solve(s, K, W)
    free.append(torch.cuda.mem_get_info()[0])
    many = _solve(s, K * copies, W * copies)
    free.append(torch.cuda.mem_get_info()[0])
    more = (free[1] - free[2]) - (free[0] - free[1])
    dE = many.energy()[0] - few.energy()[0]
    dF = np.abs(many.forces() - few.forces()).max()
    say("k-points %d on %d^3: dE %.2e dF %.2e, %.1f MB more" % (2 * copies, grid, dE, dF, more / 1e6))
    assert abs(dE) < 1e-6 * 4 and dF < 1e-4
    if grid == 48:
        assert more < 256e6 + 2 * copies * 1e6 + 16e6
