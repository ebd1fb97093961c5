// FP64 subspace solver, one workgroup per candidate up to kJacWideMax bands:
//   mode 1: orthonormalise only:  S = L L^T, M = L^-T.
//   mode 3: orthonormalise + Rayleigh-Ritz:  H' = L^-1 H L^-T = V diag(e) V^T,
//           M = L^-T V (columns sorted by ascending e), eps = e
// (the orthogonalisation and subspace-diagonalisation steps of Algorithm 1).
//
// What bounds it is latency: a chain of n elimination steps, then of (n - 1)
// Jacobi rounds per sweep, each a few hundred cycles of dependent loads and
// FP64 operations on one compute unit.  So each step is laid out for few
// instructions, one barrier (two above 64 bands), and no index arithmetic:
//  - Cholesky and W = L^-1 are one elimination on [S | I], in place (a column of
//    W takes the place of the finished column of S), with the rows in registers
//    (row i in wavefront i mod NW, a column a lane); a step publishes the pivot
//    row in LDS and takes the row multipliers by scalar lane reads;
//  - the Jacobi rounds update one triangle of H', stored by position
//    (jacobi.hpp);
//  - M's rows (those of W^T, rotated along with H') need each round's
//    rotations only: up to 32 bands other wavefronts apply them from
//    registers, a round behind; above that they are logged and applied over
//    the whole GPU afterwards (k_sub_vapply).  V and W^T V are never formed.
// Converged solves, against the same rounds on the square matrix with V in the
// loop and a Cholesky of two barriers a column: 32 bands 206 -> 103 us (a round
// 2,500 -> 1,250 cycles, the elimination 70k -> 22k cycles), 64 bands 918 -> 370
// us, 112 bands 3.27 -> 0.74 ms, 164 bands 4.58 -> 1.67 ms (a launch per round
// before); |M^T S M - 1| at 164 bands 4.8e-14 -> 5.7e-15.
#include "jacobi.hpp"
#include "launch.hpp"

#include <algorithm>
#include <mutex>

namespace sgo {

// Elimination on [S | I] in place: row i = w + NW r of wavefront w in v[r], column c
// in register c / 64, lane c mod 64.  A row below the step's k holds S in the
// columns past k and, in column c <= k, the entry of the unit-lower factor's
// inverse times -d_c (d_c: the pivot), which is what S left there: no step writes
// its own column.  S is full (both triangles).  On return v is W = L^-1.  prow:
// 2 x NQ x 64 doubles of LDS.  False (everywhere) at a pivot <= 0.
template <int NQ, int NR, int NW>
__device__ __forceinline__ bool eliminate_steps(double (&v)[NR][NQ], double (&dc)[NQ], int n, int w, int lane,
                                                double* prow) {
#pragma unroll
  for (int q = 0; q < NQ; ++q) dc[q] = 1.0;
#pragma unroll
  for (int r0 = 0; r0 < NR; ++r0) {
    const int ka = r0 * NW / 64;  // register of the step's column
    for (int kk = 0; kk < NW; ++kk) {
      const int k = r0 * NW + kk;
      if (k >= n) return true;
      double* row = prow + (k & 1) * NQ * 64;
      if (w == kk) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) row[q * 64 + lane] = v[r0][q];
      }
      __syncthreads();
      double p[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) p[q] = row[q * 64 + lane];
      const int kl = k & 63;
      const double d = readlane_d(p[ka], kl);
      if (!(d > 0.0)) return false;
      double inv = rcp_nr(d);
      inv = fma(inv, fma(-d, inv, 1.0), inv);
      dc[ka] = lane == kl ? d : dc[ka];
      p[ka] = lane == kl ? 0.0 : p[ka];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        if (r < r0 || (r == r0 && w <= kk)) continue;
        const double f = readlane_d(v[r][ka], kl) * inv;
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[r][q] = fma(-f, p[q], v[r][q]);
      }
    }
  }
  return true;
}
template <int NQ, int NR, int NW>
__device__ __forceinline__ bool eliminate(double (&v)[NR][NQ], int n, int w, int lane, double* prow) {
  double dc[NQ];  // pivots of this lane's columns
  if (!eliminate_steps<NQ, NR, NW>(v, dc, n, w, lane, prow)) return false;
  double dinv[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) dinv[q] = -1.0 / dc[q];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i = w + NW * r;
    const double f = 1.0 / sqrt(readlane_d(dc[r * NW / 64], i & 63));
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int c = q * 64 + lane;
      v[r][q] = c < i ? v[r][q] * dinv[q] * f : (c == i ? f : 0.0);
    }
  }
  return true;
}

__device__ __forceinline__ void sub_failed(const CandDesc& cd) {
  const int n = cd.nb;
  if (threadIdx.x == 0) cd.scal[S_ERR] = 2.0;
  for (int e = threadIdx.x; e < n * n; e += blockDim.x) cd.M[e] = (e / n == e % n) ? 1.0 : 0.0;
}

// Sorted eps and the ranks (ascending, ties by index) from H's diagonal.
template <bool QUAD>
__device__ __forceinline__ void jac_ranks(const CandDesc& cd, const double* T, int* rank) {
  const int n = cd.nb, n2 = n + (n & 1);
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double li = T[jac_addr<QUAD>(i, i, n2)];
    int rnk = 0;
    for (int j = 0; j < n; ++j) {
      const double lj = T[jac_addr<QUAD>(j, j, n2)];
      if (lj < li || (lj == li && j < i)) ++rnk;
    }
    rank[i] = rnk;
    cd.eps[rnk] = li;
  }
}

// The whole step for up to 8 R bands (R = 4: 32, R = 8: 64), every matrix in
// LDS or registers.  The folded work of a round: one 2x2 block of H' a lane
// (wavefronts 0 .. NH - 1), each wavefront computing the round's rotations
// itself (lane k: pair k) and reading a block's two from those lanes; the
// triangle is double-buffered, so one barrier a round.  R = 4: the other
// wavefronts rotate M's rows (4 rows to a register, 16 lanes each).
template <int R>
constexpr int sub_small_threads() { return R == 4 ? 512 : 576; }  // 9 wavefronts hold 64 bands' blocks
template <int R>
constexpr size_t sub_small_lds() {
  return sizeof(double) * (2 * (size_t)(8 * R) * (8 * R + 1) + 2 * 64 + 64);
}
template <int R>
__global__ void __launch_bounds__(sub_small_threads<R>()) k_sub_small(const CandDesc* __restrict__ cds, int mode,
                                                                      int max_sweeps) {
  const CandDesc& cd = cds[blockIdx.x];
  if (!cd.active) return;
  constexpr int N = 8 * R, LD = N + 1, TRI = N * (N + 1) / 2;
  constexpr bool inl = R == 4;  // M's rows rotated here
  const int n = cd.nb, n2 = n + (n & 1), np = n2 / 2, m = n2 - 1;
  const int tid = threadIdx.x, lane = tid & 63, W = blockDim.x >> 6;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  extern __shared__ __align__(16) char smem[];
  double* Hl = (double*)smem;      // H, then the two triangles of H'
  double* Wl = Hl + N * LD;        // W = L^-1
  double* prow = Wl + N * LD;      // pivot rows
  double2* cs = (double2*)(prow + 2 * 64);  // rotations of two rounds (R = 4)
  __shared__ double sh[16 * 2];
  __shared__ int rank_l[N];
  long long* clk = cd.dbg_clk;
  if (clk && tid == 0) clk[0] = clock64();
  if (mode == 3)
    for (int u = w; u < n; u += W)
      if (lane < n) Hl[u * LD + lane] = 0.5 * (cd.Hs[u * n + lane] + cd.Hs[lane * n + u]);
  // rows of S (from its lower triangle), then of W
  double v[R][1];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = w + 8 * r;
    const bool in = w < 8 && i < n && lane < n;
    v[r][0] = in ? cd.S[max(i, lane) * n + min(i, lane)] : 0.0;
  }
  if (!eliminate<1, R, 8>(v, n, w, lane, prow)) {
    sub_failed(cd);
    return;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = w + 8 * r;
    if (w < 8 && i < n && lane < n) Wl[i * LD + lane] = v[r][0];
  }
  __syncthreads();
  if (clk && tid == 0) clk[1] = clock64();
  if (mode == 1) {
    for (int u = w; u < n; u += W)
      if (lane < n) cd.M[u * n + lane] = Wl[lane * LD + u];
    return;
  }
  // H' = W H W^T: the wavefront's rows of T = W H, then of T W^T, a column a lane
  double t[R], h[R];
#pragma unroll
  for (int r = 0; r < R; ++r) t[r] = h[r] = 0.0;
  if (w < 8) {
    for (int k = 0; k < n; ++k) {
      const double hk = Hl[k * LD + min(lane, N - 1)];
#pragma unroll
      for (int r = 0; r < R; ++r) t[r] = fma(readlane_d(v[r][0], k), hk, t[r]);
    }
    for (int k = 0; k < n; ++k) {
      const double wk = Wl[min(lane, N - 1) * LD + k];
#pragma unroll
      for (int r = 0; r < R; ++r) h[r] = fma(readlane_d(t[r], k), wk, h[r]);
    }
  }
  __syncthreads();  // H is read
  double* T = Hl;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = w + 8 * r;
    if (w < 8 && i < n && lane <= i) T[jac_addr<false>(i, lane, n2)] = h[r];
  }
  if (n2 > n && w == 0 && lane <= n) T[jac_addr<false>(n, lane, n2)] = 0.0;
  __syncthreads();
  if (clk && tid == 0) clk[2] = clock64();
  const int nblk = np * (np + 1) / 2, NH = (nblk + 63) / 64;
  // this lane's block
  JacBlock blk;
  const bool on = w * 64 + lane < nblk;
  blk.init<false>(min(w * 64 + lane, nblk - 1), n2);
  const int k = min(lane, np - 1);
  const int ia = jac_addr<false>(k, k, n2), ib = jac_addr<false>(n2 - 1 - k, n2 - 1 - k, n2), ic = jac_addr<false>(n2 - 1 - k, k, n2);
  const int pP = 4 * blk.P, pQ = 4 * blk.Q;
  const bool diag = blk.P == blk.Q;
  // this lane's entries of M's rows: row j starts as row j of W^T
  constexpr int SETS = 2;
  const int kv = lane & 15;
  const bool is0 = kv == 0, is_last = kv == np - 1;
  double vt[SETS] = {0.0, 0.0}, vb[SETS] = {0.0, 0.0};
  int nsets = 0;
  if (inl && w >= NH) {
    const int wv = w - NH, Wv = W - NH, tot = (n + 3) / 4;
    nsets = wv < tot ? (tot - wv + Wv - 1) / Wv : 0;
#pragma unroll
    for (int q = 0; q < SETS; ++q) {
      const int j = (wv + q * Wv) * 4 + (lane >> 4), ibot = n2 - 1 - kv;
      vt[q] = j < n && kv < np ? Wl[kv * LD + j] : 0.0;
      vb[q] = j < n && kv < np && ibot < n ? Wl[ibot * LD + j] : 0.0;
    }
  }
  double2* log = (double2*)(cd.red_part + kJacLog);
  int par = 0, nsweep = 0;
  bool pending = false;
  const int limit = n > 1 ? max_sweeps : 0;
  for (int sweep = 0; sweep < limit; ++sweep) {
    if (jac_converged<false>(T + par * TRI, n2, sh)) break;
    ++nsweep;
    for (int r = 0; r < m; ++r) {
      if (w < NH) {
        const double* A = T + par * TRI;
        double* B = T + (TRI - par * TRI);
        const double app = A[ia], aqq = A[ib], apq = A[ic];
        double x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = A[blk.rd[q]];
        double c, s;
        jac_rotation(app, aqq, apq, k, n2 - 1 - k, r, m, &c, &s);
        const double cP = bperm_d(pP, c), sP = bperm_d(pP, s), cQ = bperm_d(pQ, c), sQ = bperm_d(pQ, s);
        if (w == 0 && lane < np) {
          if (inl) cs[par * 16 + lane] = make_double2(c, s);
          else log[(size_t)(sweep * m + r) * np + lane] = make_double2(c, s);
        }
        jac_block_update(x, cP, sP, cQ, sQ, diag);
        if (on) {
#pragma unroll
          for (int q = 0; q < 4; ++q) B[blk.wr[q]] = x[q];
        }
      } else if (inl && pending && nsets > 0) {
        const double2 z = cs[(par ^ 1) * 16 + kv];
        jac_row_step(vt[0], vb[0], z.x, z.y, is0, is_last);
        if (nsets > 1) jac_row_step(vt[1], vb[1], z.x, z.y, is0, is_last);
      }
      pending = true;
      par ^= 1;
      __syncthreads();
    }
  }
  if (inl && pending && nsets > 0) {
    const double2 z = cs[(par ^ 1) * 16 + kv];
    jac_row_step(vt[0], vb[0], z.x, z.y, is0, is_last);
    if (nsets > 1) jac_row_step(vt[1], vb[1], z.x, z.y, is0, is_last);
  }
  if (clk && tid == 0) {
    clk[3] = clock64();
    clk[5] = nsweep;
  }
  int* rank = inl ? rank_l : (int*)(cd.red_part + kJacRanks);
  jac_ranks<false>(cd, T + par * TRI, rank);
  if (inl) {
    __syncthreads();
    const int wv = w - NH, Wv = W - NH, ibot = n2 - 1 - kv;
#pragma unroll
    for (int q = 0; q < SETS; ++q) {
      const int j = (wv + q * Wv) * 4 + (lane >> 4);
      if (q < nsets && j < n && kv < np) {
        cd.M[j * n + rank[kv]] = vt[q];
        if (ibot < n) cd.M[j * n + rank[ibot]] = vb[q];
      }
    }
  } else {  // W and the log go to k_sub_vapply
    for (int u = w; u < n; u += W)
      if (lane < n) cd.C[u * n + lane] = Wl[u * LD + lane];
    if (tid == 0) cd.red_part[kJacSweeps] = nsweep;
  }
  if (clk && tid == 0) clk[4] = clock64();
}

// Cholesky and W = L^-1 (into C) above 64 bands: the same elimination, 16
// wavefronts, NR rows and NQ columns a lane (<2, 8>: 128, <3, 12>: 192, <4, 13>:
// 208; the last keeps 13 registers in scratch memory).  112 bands 56 us; 164 bands
// 119 us, 435 us by blocks of rows in global memory; 198 bands with M = W^T 192 us,
// 539 us.
template <int NQ, int NR>
__global__ void __launch_bounds__(1024) k_sub_chol(const CandDesc* __restrict__ cds) {
  const CandDesc& cd = cds[blockIdx.x];
  if (!cd.active) return;
  constexpr int NW = 16;
  const int n = cd.nb, lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __shared__ double prow[2 * NQ * 64];
  long long* clk = cd.dbg_clk;
  if (clk && threadIdx.x == 0) clk[0] = clock64();
  double v[NR][NQ];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i = w + NW * r;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int c = q * 64 + lane;
      v[r][q] = i < n && c < n ? cd.S[(size_t)max(i, c) * n + min(i, c)] : 0.0;
    }
  }
  if (!eliminate<NQ, NR, NW>(v, n, w, lane, prow)) {
    sub_failed(cd);
    return;
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i = w + NW * r;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int c = q * 64 + lane;
      if (i < n && c < n) cd.C[(size_t)i * n + c] = v[r][q];
    }
  }
  if (clk && threadIdx.x == 0) clk[1] = clock64();
}
// M = W^T (mode 1 above 64 bands)
__global__ void __launch_bounds__(kNT) k_sub_wt(const CandDesc* __restrict__ cds) {
  const CandDesc& cd = cds[blockIdx.y];
  if (!cd.active || cd.scal[S_ERR] == 2.0) return;
  const int n = cd.nb, e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n * n) cd.M[e] = cd.C[(size_t)(e % n) * n + e / n];
}

// The Jacobi rounds of 65 to kJacWideMax bands: H' (formed over the GPU, in Hs)
// in LDS, once; ITEMS blocks a thread, read into registers before the round's
// first write.  Lanes 0 .. np - 1 of the workgroup compute the rotations and
// publish them in LDS (computed in every wavefront they would cost more
// issue slots than the blocks): two barriers a round.  The log goes to
// k_sub_vapply: M's rows would be two thirds of a round's work on the one
// compute unit that the chain keeps busy.
template <int ITEMS>
__global__ void __launch_bounds__(1024) k_sub_jacobi(const CandDesc* __restrict__ cds, int max_sweeps) {
  const CandDesc& cd = cds[blockIdx.x];
  if (!cd.active || cd.scal[S_ERR] == 2.0) return;  // inactive, or a Cholesky failed
  const int n = cd.nb, n2 = n + (n & 1), np = n2 / 2, m = n2 - 1;
  const int nblk = np * (np + 1) / 2, nt = n2 * (n2 + 1) / 2;
  const int tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  extern __shared__ __align__(16) char smem[];
  double2* cs = (double2*)smem;      // [np]
  double* T = (double*)(cs + np);    // [nt], then a slot for the idle lanes' writes
  __shared__ double sh[16 * 2];
  for (int u = tid >> 6; u < n2; u += nthr >> 6)
    for (int v = lane; v <= u; v += 64) T[jac_addr<true>(u, v, n2)] = u < n ? cd.Hs[(size_t)u * n + v] : 0.0;
  if (cd.dbg_clk && tid == 0) cd.dbg_clk[2] = clock64();
  int rd[ITEMS][4], wr[ITEMS][4], P[ITEMS], Q[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int t = tid + i * nthr;
    JacBlock b;
    b.init<true>(min(t, nblk - 1), n2);
    P[i] = b.P;
    Q[i] = b.Q;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      rd[i][q] = b.rd[q];
      wr[i][q] = t < nblk ? b.wr[q] : nt;
    }
  }
  const int k = min(tid, np - 1);
  const int ia = jac_addr<true>(k, k, n2), ib = jac_addr<true>(n2 - 1 - k, n2 - 1 - k, n2), ic = jac_addr<true>(n2 - 1 - k, k, n2);
  double2* log = (double2*)(cd.red_part + kJacLog);
  __syncthreads();
  int nsweep = 0;
  const int limit = n > 1 ? max_sweeps : 0;
  for (int sweep = 0; sweep < limit; ++sweep) {
    if (jac_converged<true>(T, n2, sh)) break;
    ++nsweep;
    for (int r = 0; r < m; ++r) {
      if ((tid & ~63) < np) {  // uniform per wavefront
        double c, s;
        jac_rotation(T[ia], T[ib], T[ic], k, n2 - 1 - k, r, m, &c, &s);
        if (tid < np) {
          const double2 z = make_double2(c, s);
          cs[tid] = z;
          log[(size_t)(sweep * m + r) * np + tid] = z;
        }
      }
      double x[ITEMS][4];
#pragma unroll
      for (int i = 0; i < ITEMS; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) x[i][q] = T[rd[i][q]];
      __syncthreads();  // rotations published, every entry of the round read
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        const double2 zp = cs[P[i]], zq = cs[Q[i]];
        jac_block_update(x[i], zp.x, zp.y, zq.x, zq.y, P[i] == Q[i]);
#pragma unroll
        for (int q = 0; q < 4; ++q) T[wr[i][q]] = x[i][q];
      }
      __syncthreads();
    }
  }
  jac_ranks<true>(cd, T, (int*)(cd.red_part + kJacRanks));
  if (tid == 0) {
    cd.red_part[kJacSweeps] = nsweep;
    if (cd.dbg_clk) {
      cd.dbg_clk[3] = cd.dbg_clk[4] = clock64();
      cd.dbg_clk[5] = nsweep;
    }
  }
}

// M = W^T V from the logged rotations: one wavefront per row of M, which
// starts as the row of W^T (in C) and takes each round's rotations on its
// lanes' pairs (SETS of 64).
constexpr int kVapplyAhead = 4;  // rounds whose rotations are loaded ahead
template <int SETS>
__global__ void __launch_bounds__(kNT) k_sub_vapply(const CandDesc* __restrict__ cds) {
  const CandDesc& cd = cds[blockIdx.y];
  if (!cd.active || cd.scal[S_ERR] == 2.0) return;
  const int n = cd.nb, n2 = n + (n & 1), np = n2 / 2, lane = threadIdx.x & 63;
  const int j = blockIdx.x * (kNT / 64) + (threadIdx.x >> 6);
  if (j >= n) return;
  const double2* log = (const double2*)(cd.red_part + kJacLog);
  const int rounds = (int)cd.red_part[kJacSweeps] * (n2 - 1);
  double vt[SETS], vb[SETS];
  int kk[SETS];
#pragma unroll
  for (int q = 0; q < SETS; ++q) {
    const int k = q * 64 + lane;
    kk[q] = min(k, np - 1);
    vt[q] = k < np ? cd.C[(size_t)k * n + j] : 0.0;
    vb[q] = k < np && n2 - 1 - k < n ? cd.C[(size_t)(n2 - 1 - k) * n + j] : 0.0;
  }
  double2 z[kVapplyAhead][SETS];
#pragma unroll
  for (int u = 0; u < kVapplyAhead; ++u)
#pragma unroll
    for (int q = 0; q < SETS; ++q)
      if (u < rounds) z[u][q] = log[(size_t)u * np + kk[q]];
  for (int r0 = 0; r0 < rounds; r0 += kVapplyAhead) {
#pragma unroll
    for (int u = 0; u < kVapplyAhead; ++u) {
      if (r0 + u >= rounds) break;
      double t[SETS], b[SETS];
#pragma unroll
      for (int q = 0; q < SETS; ++q) {
        const double c = z[u][q].x, s = z[u][q].y;
        t[q] = fma(c, vt[q], -(s * vb[q]));
        b[q] = fma(s, vt[q], c * vb[q]);
        if (r0 + u + kVapplyAhead < rounds) z[u][q] = log[(size_t)(r0 + u + kVapplyAhead) * np + kk[q]];
      }
#pragma unroll
      for (int q = 0; q < SETS; ++q) {
        const int k = q * 64 + lane;
        double tn = dpp_d<kDppWaveShl1>(t[q]), bn = dpp_d<kDppWaveShr1>(b[q]);
        if (q + 1 < SETS) {
          const double x = readlane_d(t[q + 1 < SETS ? q + 1 : 0], 0);
          if (lane == 63) tn = x;
        }
        if (q > 0) {
          const double x = readlane_d(b[q > 0 ? q - 1 : 0], 63);
          if (lane == 0) bn = x;
        }
        const bool is0 = k == 0, is_last = k == np - 1;
        const double x = is_last ? b[q] : tn;
        vt[q] = is0 ? t[q] : x;
        vb[q] = is0 ? x : bn;
      }
    }
  }
  const int* rank = (const int*)(cd.red_part + kJacRanks);
#pragma unroll
  for (int q = 0; q < SETS; ++q) {
    const int k = q * 64 + lane;
    if (k < np) {
      cd.M[(size_t)j * n + rank[k]] = vt[q];
      if (n2 - 1 - k < n) cd.M[(size_t)j * n + rank[n2 - 1 - k]] = vb[q];
    }
  }
}

// ---------------------------------------------------------------- launchers
static void launch_vapply(hipStream_t st, const CandDesc* desc, int ncand, int n) {
  const dim3 gv((n + kNT / 64 - 1) / (kNT / 64), ncand);
  if (n <= 128) hipLaunchKernelGGL(k_sub_vapply<1>, gv, dim3(kNT), 0, st, desc);
  else hipLaunchKernelGGL(k_sub_vapply<2>, gv, dim3(kNT), 0, st, desc);
  check_launch("k_sub_vapply");
}

template <int ITEMS>
static void launch_rounds(hipStream_t st, const CandDesc* desc, int ncand, int n, int max_sweeps) {
  const int n2 = n + (n & 1), np = n2 / 2, nblk = np * (np + 1) / 2;
  // as few wavefronts as hold the blocks in equal shares
  const int waves = (nblk + 64 * ITEMS - 1) / (64 * ITEMS);
  const size_t lds = sizeof(double) * ((size_t)n2 * (n2 + 1) / 2 + 1 + 2 * np);
  hipLaunchKernelGGL(k_sub_jacobi<ITEMS>, dim3(ncand), dim3(64 * waves), lds, st, desc, max_sweeps);
  check_launch("k_sub_jacobi");
}

// No host sync and no allocation: this serves graph capture and the
// allocation-free entry point too.
void launch_sub_block(hipStream_t st, const CandDesc* desc, int ncand, int n, int mode, int max_sweeps) {
  max_sweeps = std::min(max_sweeps, kJacMaxSweeps);  // the log holds no more
  if (n <= 32) {
    hipLaunchKernelGGL(k_sub_small<4>, dim3(ncand), dim3(sub_small_threads<4>()), sub_small_lds<4>(), st, desc,
                       mode, max_sweeps);
    check_launch("k_sub_small");
    return;
  }
  if (n <= 64) {
    hipLaunchKernelGGL(k_sub_small<8>, dim3(ncand), dim3(sub_small_threads<8>()), sub_small_lds<8>(), st, desc,
                       mode, max_sweeps);
    check_launch("k_sub_small");
    if (mode == 3) launch_vapply(st, desc, ncand, n);
    return;
  }
  if (n <= 128) hipLaunchKernelGGL((k_sub_chol<2, 8>), dim3(ncand), dim3(1024), 0, st, desc);
  else if (n <= 192) hipLaunchKernelGGL((k_sub_chol<3, 12>), dim3(ncand), dim3(1024), 0, st, desc);
  else hipLaunchKernelGGL((k_sub_chol<4, 13>), dim3(ncand), dim3(1024), 0, st, desc);
  check_launch("k_sub_chol");
  if (mode == 1) {
    hipLaunchKernelGGL(k_sub_wt, dim3((n * n + kNT - 1) / kNT, ncand), dim3(kNT), 0, st, desc);
    check_launch("k_sub_wt");
    return;
  }
  launch_sub_congruence(st, desc, ncand, n);
  const int np = (n + 1) / 2, nblk = np * (np + 1) / 2;
  switch ((nblk + 1023) / 1024) {
    case 1: launch_rounds<1>(st, desc, ncand, n, max_sweeps); break;
    case 2: launch_rounds<2>(st, desc, ncand, n, max_sweeps); break;
    case 3: launch_rounds<3>(st, desc, ncand, n, max_sweeps); break;
    case 4: launch_rounds<4>(st, desc, ncand, n, max_sweeps); break;
    default: launch_rounds<5>(st, desc, ncand, n, max_sweeps); break;
  }
  launch_vapply(st, desc, ncand, n);
}

void configure_sub_kernels() {
  allow_lds((const void*)k_sub_small<4>);
  allow_lds((const void*)k_sub_small<8>);
  allow_lds((const void*)k_sub_jacobi<1>);
  allow_lds((const void*)k_sub_jacobi<2>);
  allow_lds((const void*)k_sub_jacobi<3>);
  allow_lds((const void*)k_sub_jacobi<4>);
  allow_lds((const void*)k_sub_jacobi<5>);
}

}  // namespace sgo
