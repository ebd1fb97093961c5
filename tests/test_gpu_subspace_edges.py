"""The subspace step at the edges of its kernels' size ranges, allocating and
allocation-free: S-orthonormal bands, a diagonal H, ascending eigenvalues.

Ranges: 32 and 64 bands (matrices in LDS), 128 (row elimination), 198
(one-workgroup Jacobi rounds), the block counts at which a thread takes one
more block (np (np + 1) / 2 over 1024), odd and even.  Tolerance: a solve is
at most about 10 sweeps of n rounds of rotations orthogonal to 2 ulp, so
10 n 4e-16 < 1e-12 at every size, times a margin of 4 for the products."""
import numpy as np
import pytest

import paper_1603_02732_amd as sgo

pytestmark = pytest.mark.gpu
TOL = 4e-12


def _problem(n, kind):
    rng = np.random.default_rng(n)
    A = rng.normal(size=(n, n)) / np.sqrt(n)
    S = np.eye(n) + 0.1 * (A + A.T)
    if kind == "ties":  # every diagonal difference of the first round is zero
        return np.eye(n), 0.01 * np.ones((n, n)) + np.eye(n)
    B = rng.normal(size=(n, n)) / np.sqrt(n)
    return S, np.diag(np.sort(rng.uniform(-1, 1, n))) + 0.2 * (B + B.T)


def _noalloc(S, H, mode):
    import torch
    n = len(S)
    tS, tH = torch.from_numpy(S).cuda(), torch.from_numpy(H).cuda()
    M = torch.full((n, n), float("nan"), dtype=torch.float64, device="cuda")
    e = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    sgo.subspace_solve_noalloc(tS.data_ptr(), tH.data_ptr(), M.data_ptr(), e.data_ptr(), n, mode,
                               stream=torch.cuda.current_stream().cuda_stream)
    return M.cpu().numpy(), e.cpu().numpy()


def _check(S, H, M, e):
    n = len(S)
    print("n=%d orth %.1e diag %.1e" % (n, np.abs(M.T @ S @ M - np.eye(n)).max(),
                                        np.abs(M.T @ H @ M - np.diag(e)).max()), flush=True)
    assert np.abs(M.T @ S @ M - np.eye(n)).max() < TOL
    assert np.abs(M.T @ H @ M - np.diag(e)).max() < TOL
    assert (np.diff(e) >= 0).all()
    L = np.linalg.inv(np.linalg.cholesky(S))
    assert np.abs(np.linalg.eigvalsh(L @ H @ L.T) - e).max() < TOL


SIZES = [1, 2, 3, 16, 17, 31, 32, 33, 63, 64, 65, 88, 89, 90, 126, 127, 128, 129, 154, 157, 180,
         181, 197, 198, 199]


@pytest.mark.parametrize("n", SIZES)
def test_both_forms_at_the_edges(n):
    S, H = _problem(n, "random")
    M, e, _, _ = sgo.subspace_solve(S, H, mode=3)
    _check(S, H, M, e)
    M, e = _noalloc(S, H, 3)
    _check(S, H, M, e)
    M1, _ = _noalloc(S, H, 1)
    assert np.abs(M1 - np.linalg.inv(np.linalg.cholesky(S)).T).max() < TOL


@pytest.mark.parametrize("n", [8, 33, 66, 130])
def test_equal_diagonals(n):
    S, H = _problem(n, "ties")
    M, e = _noalloc(S, H, 3)
    _check(S, H, M, e)


@pytest.mark.parametrize("n", [200, 224, 255, 256])
def test_largest_without_allocation(n):
    S, H = _problem(n, "random")
    M, e = _noalloc(S, H, 3)
    _check(S, H, M, e)


@pytest.mark.parametrize("n", [24, 48, 112, 198, 224])
def test_captured(n):
    """The allocation-free step in a HIP graph: every route is launches alone, and
    each replay, on new matrices and with eager calls in between, gives the
    eager bits."""
    import torch
    probs = [_problem(n, "random")]
    probs.append((probs[0][0] + 0.01 * np.eye(n), probs[0][1][::-1, ::-1].copy()))
    eager = [_noalloc(S, H, 3) for S, H in probs]
    dev = [[torch.from_numpy(x).cuda() for x in p] for p in probs]
    S, H = dev[0][0].clone(), dev[0][1].clone()
    M, e = torch.zeros(n, n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    st = torch.ones(1, dtype=torch.int32, device="cuda")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        sgo.subspace_solve_noalloc(S.data_ptr(), H.data_ptr(), M.data_ptr(), e.data_ptr(), n, 3,
                                   status=st.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
    for k in (0, 1, 0, 1):
        print("n=%d replay on matrices %d" % (n, k), flush=True)
        S.copy_(dev[k][0])
        H.copy_(dev[k][1])
        M.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        assert np.array_equal(M.cpu().numpy(), eager[k][0]) and np.array_equal(e.cpu().numpy(), eager[k][1])
        _noalloc(*probs[1 - k], 3)


@pytest.mark.parametrize("mode", [1, 3])
@pytest.mark.parametrize("n", [20, 40, 100, 150, 198, 200])
def test_not_positive_definite(n, mode):
    """Every Cholesky: up to 32, 64, 128, 192 and 198 bands in registers, above
    in panels; the bad pivot first, in the middle and last.  The status says so,
    M is the identity, the inputs stay, and the next call is not affected."""
    import torch
    S, H = _problem(n, "random")
    tH = torch.from_numpy(H).cuda()
    e = torch.zeros(n, dtype=torch.float64, device="cuda")
    for bad in (0, n // 2, n - 1):
        print("n=%d mode=%d bad pivot %d" % (n, mode, bad), flush=True)
        B = S.copy()
        B[bad, bad] = -1.0
        tS = torch.from_numpy(B).cuda()
        M = torch.full((n, n), float("nan"), dtype=torch.float64, device="cuda")
        st = torch.zeros(1, dtype=torch.int32, device="cuda")
        sgo.subspace_solve_noalloc(tS.data_ptr(), tH.data_ptr(), M.data_ptr(), e.data_ptr(), n, mode,
                                   status=st.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
        assert int(st.item()) == sgo.SGO_ENUMERIC
        assert np.array_equal(M.cpu().numpy(), np.eye(n))
        assert np.array_equal(tS.cpu().numpy(), B) and np.array_equal(tH.cpu().numpy(), H)
        with pytest.raises(sgo.SgoError) as err:
            sgo.subspace_solve(B, H, mode=mode)
        assert err.value.code == sgo.SGO_ENUMERIC
        M, _ = _noalloc(S, H, mode)
        assert np.abs(M.T @ S @ M - np.eye(n)).max() < TOL
