// k-point sampling of the Brillouin zone (the rough k-point grids that
// Section 2.3 allows for the energy evaluations of a search): FP64 kernels
// of the complex-band path.  At a k-point the Bloch periodic parts
// u_nk = sum_G c_G e^{iG.r} live on the shifted sphere |k+G|^2/2 <= Ecut,
// complex with no relation between c(G) and c(-G), so one band is one
// complex FFT (no pairing of two real bands) and every subspace matrix is
// complex Hermitian.  Bands are rows X[band][npw] of complex coefficients.
// The steps are those of Algorithm 1 (H psi, subspace matrix, Cholesky
// orthonormalisation, subspace diagonalisation, residual, preconditioned
// CG direction, projection, line minimisation) for each k, and the density
// of Section 2.4 summed over k with the k-point weights.  The grid side
// (mixing, potentials, energies) is the Gamma path's.
//
// A rough mesh has a few k-points of a small cell, so a launch is a few
// microseconds of work: every launch covers all k-points (a descriptor per k),
// H psi of a band is one workgroup with its grid in LDS, and the subspace step
// one workgroup per k.  8 silicon atoms, 15^3, 20 bands, 2 k-points: 3,130
// launches and 110 ms per solve with a launch per k, pass and array and one
// 256-thread workgroup walking the Jacobi pairs of a k in turn, 790 launches and
// 10.1 ms this way (other positions take 8 to 13 ms, by their iterations).
#include "device.hpp"
#include "fft_lds.hpp"
#include "jacobi.hpp"
#include "launch.hpp"

#include <algorithm>

namespace sgo {

using zc = cplx<double>;

__device__ __forceinline__ zc zconj(zc a) { return {a.x, -a.y}; }
__device__ __forceinline__ zc zmul(zc a, zc b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
// conj(a) b
__device__ __forceinline__ zc zcmul(zc a, zc b) { return {a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x}; }
__device__ __forceinline__ zc zscale(zc a, double s) { return {a.x * s, a.y * s}; }
__device__ __forceinline__ zc zadd(zc a, zc b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ zc zsub(zc a, zc b) { return {a.x - b.x, a.y - b.y}; }
// a + b c
__device__ __forceinline__ zc zfma(zc b, zc c, zc a) {
  return {fma(b.x, c.x, fma(-b.y, c.y, a.x)), fma(b.x, c.y, fma(b.y, c.x, a.y))};
}

__device__ __forceinline__ zc* band_array(const KptDev& k, int which) {
  switch (which) {
    case W_X: return k.X;
    case W_HX: return k.HX;
    case W_D: return k.D;
    case W_HD: return k.HD;
    default: return k.beta;
  }
}

// ------------------------------------------------------------------ grids
__global__ void k_kpt_zero(zc* __restrict__ a, long n) {
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x)
    a[e] = {0.0, 0.0};
}

// z[b][box[g]] = src[b][g]
__global__ void k_kpt_scatter(const KptDev* __restrict__ kd, zc* __restrict__ z, int src, long ntot) {
  const KptDev& k = kd[blockIdx.y];
  const zc* X = band_array(k, src);
  zc* zk = z + (size_t)blockIdx.y * k.nb * ntot;
  const long n = (long)k.nb * k.npw;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    const int b = (int)(e / k.npw), g = (int)(e - (long)b * k.npw);
    zk[(long)b * ntot + k.box[g]] = X[e];
  }
}

// Batched line transforms along one axis of grids [nb][N3][N2][N1]: line l
// starts at (l / A) * Bs + (l % A) * Cs and its elements are es apart.  L
// lines per workgroup go through LDS together (fft_lds.hpp).
__global__ void __launch_bounds__(256) k_kpt_lines(zc* __restrict__ data, FftPlan P, int A, long Bs,
                                                   long Cs, long es, long nlines, int L, int sign) {
  extern __shared__ __align__(16) char smem[];
  const int n = P.n, p = n | 1, tid = threadIdx.x, nthr = blockDim.x;
  zc* a = (zc*)smem;
  zc* tw = a + (size_t)L * p;
  unsigned char* pos = (unsigned char*)(tw + n);
  lds_tables<double>(tw, nullptr, pos, P, 192);
  const long l0 = (long)blockIdx.x * L;
  const int nl = (int)min((long)L, nlines - l0);
  for (int t = tid; t < nl * n; t += nthr) {
    // consecutive threads take consecutive memory: along the line (es == 1)
    // or across lines
    int l, e;
    if (es == 1) {
      l = t / n;
      e = t - l * n;
    } else {
      e = t / nl;
      l = t - e * nl;
    }
    const long line = l0 + l;
    a[l * p + e] = data[(line / A) * Bs + (line % A) * Cs + e * es];
  }
  __syncthreads();
  lds_dif<double>(a, {nl, p, 1, nl, 0}, P, tw, (double)sign);
  for (int t = tid; t < nl * n; t += nthr) {
    int l, e;
    if (es == 1) {
      l = t / n;
      e = t - l * n;
    } else {
      e = t / nl;
      l = t - e * nl;
    }
    const long line = l0 + l;
    data[(line / A) * Bs + (line % A) * Cs + e * es] = a[l * p + pos[e]];
  }
}

// z[b][r] *= V(r)
__global__ void k_kpt_vmul(zc* __restrict__ zk, const double* __restrict__ v, int nb, long ntot) {
  const long n = (long)nb * ntot;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x)
    zk[e] = zscale(zk[e], v[e % ntot]);
}

// dst[b][g] = |k+G|^2/2 src[b][g] + z[b][box[g]] / ntot
__global__ void k_kpt_gather(const KptDev* __restrict__ kd, const zc* __restrict__ z, int src, int dst,
                             long ntot) {
  const KptDev& k = kd[blockIdx.y];
  const zc* X = band_array(k, src);
  zc* Y = band_array(k, dst);
  const zc* zk = z + (size_t)blockIdx.y * k.nb * ntot;
  const long n = (long)k.nb * k.npw;
  const double s = 1.0 / (double)ntot;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    const int b = (int)(e / k.npw), g = (int)(e - (long)b * k.npw);
    const zc w = zk[(long)b * ntot + k.box[g]];
    Y[e] = {k.kin[g] * X[e].x + w.x * s, k.kin[g] * X[e].y + w.y * s};
  }
}

// --------------------------------------------- small grids, in LDS
struct KGrid {
  int N1, N2, N3;
};
// One axis of the LDS grid [N3][N2][N1 | 1]: line l starts at (l / A) B + (l % A)
// C, elements es apart.  One thread transforms a line in its registers: e^{+i}
// with sg = 1, e^{-i} (the conjugate of the transform of the conjugate) with -1.
template <int N>
__device__ __forceinline__ void grid_lines(zc* g, int nlines, int A, int B, int C, int es, double sg) {
  for (int l = threadIdx.x; l < nlines; l += blockDim.x) {
    zc* p = g + (l / A) * B + (l % A) * C;
    zc in[N], out[N];
#pragma unroll
    for (int j = 0; j < N; ++j) in[j] = {p[j * es].x, sg * p[j * es].y};
    freg::fft<double, 1, N>(in, out);
#pragma unroll
    for (int j = 0; j < N; ++j) p[j * es] = {out[j].x, sg * out[j].y};
  }
}
// The grid to r (z, y, x) and, given v, times v and back (x, y, z): one copy of
// the line code.  NM: the longest line of the launch (16, 20 or 32), which
// sets the registers.
template <int NM>
__device__ __forceinline__ void grid_transform(zc* g, const KGrid& K, const double* v) {
  const int p = K.N1 | 1, ntot = K.N1 * K.N2 * K.N3;
  for (int step = 0; step < (v ? 6 : 3); ++step) {
    if (step == 3) {
      for (int e = threadIdx.x; e < ntot; e += blockDim.x) {
        const int row = e / K.N1, q = row * p + e - row * K.N1;
        g[q] = zscale(g[q], v[e]);
      }
      __syncthreads();
    }
    const int ax = step < 3 ? 2 - step : step - 3;
    const double sg = step < 3 ? 1.0 : -1.0;
    const int N = ax == 0 ? K.N1 : (ax == 1 ? K.N2 : K.N3);
    const int nlines = ax == 0 ? K.N2 * K.N3 : (ax == 1 ? p * K.N3 : p * K.N2);
    const int A = ax == 0 ? 1 : (ax == 1 ? p : p * K.N2);
    const int B = ax == 0 ? p : (ax == 1 ? p * K.N2 : 0);
    const int C = ax == 0 ? 0 : 1;
    const int es = ax == 0 ? 1 : (ax == 1 ? p : p * K.N2);
    switch (N) {
#define SGO_LINE(n)                                                                     \
  case n:                                                                               \
    if constexpr (n <= NM) grid_lines<n>(g, nlines, A, B, C, es, sg);                   \
    break;
      SGO_LINE(1) SGO_LINE(2) SGO_LINE(3) SGO_LINE(4) SGO_LINE(5) SGO_LINE(6) SGO_LINE(8) SGO_LINE(9)
      SGO_LINE(10) SGO_LINE(12) SGO_LINE(15) SGO_LINE(16) SGO_LINE(18) SGO_LINE(20) SGO_LINE(24)
      SGO_LINE(25) SGO_LINE(27) SGO_LINE(30) SGO_LINE(32)
#undef SGO_LINE
    }
    __syncthreads();
  }
}
__device__ __forceinline__ void grid_fill(zc* g, const KGrid& K, const zc* x, const int* box, int npw) {
  const int p = K.N1 | 1;
  for (int e = threadIdx.x; e < p * K.N2 * K.N3; e += blockDim.x) g[e] = {0.0, 0.0};
  __syncthreads();
  for (int i = threadIdx.x; i < npw; i += blockDim.x) {
    const int row = box[i] / K.N1;
    g[row * p + box[i] - row * K.N1] = x[i];
  }
  __syncthreads();
}

// (kinetic + V) src -> dst of one band of one k: the whole grid in LDS.  Bound
// by the latency of its six transform passes (nlines of them on 256 threads);
// 2 x 20 bands of 15^3: 14.5 us, where the 10 launches of the pass-by-pass
// route take 96 us.
template <int NM>
__global__ void __launch_bounds__(256) k_kpt_hpsi(const KptDev* __restrict__ kd, KGrid K, int src, int dst,
                                                  const double* __restrict__ veff) {
  const KptDev& k = kd[blockIdx.y];
  extern __shared__ __align__(16) char smem[];
  zc* g = (zc*)smem;
  const int npw = k.npw, p = K.N1 | 1, ntot = K.N1 * K.N2 * K.N3;
  const zc* x = band_array(k, src) + (size_t)blockIdx.x * npw;
  zc* y = band_array(k, dst) + (size_t)blockIdx.x * npw;
  const int* box = k.box;
  const double* kin = k.kin;
  grid_fill(g, K, x, box, npw);
  grid_transform<NM>(g, K, veff);
  const double s = 1.0 / ntot;
  for (int i = threadIdx.x; i < npw; i += blockDim.x) {
    const int row = box[i] / K.N1;
    const zc w = g[row * p + box[i] - row * K.N1];
    y[i] = {kin[i] * x[i].x + w.x * s, kin[i] * x[i].y + w.y * s};
  }
}

// part[(ik nchunk + chunk)][r] = w_k sum over the chunk's bands f_n |u_n(r)|^2
template <int NM>
__global__ void __launch_bounds__(256) k_kpt_dens_lds(const KptDev* __restrict__ kd, KGrid K, int nchunk,
                                                      double* __restrict__ part) {
  const KptDev& k = kd[blockIdx.y];
  extern __shared__ __align__(16) char smem[];
  const int p = K.N1 | 1, ntot = K.N1 * K.N2 * K.N3;
  zc* g = (zc*)smem;
  double* o = part + ((size_t)blockIdx.y * nchunk + blockIdx.x) * ntot;
  for (int e = threadIdx.x; e < ntot; e += blockDim.x) o[e] = 0.0;
  for (int b = blockIdx.x; b < k.nb; b += nchunk) {
    const double f = k.w * k.occ[b];
    if (f == 0.0) continue;  // the same for every thread
    grid_fill(g, K, k.X + (size_t)b * k.npw, k.box, k.npw);
    grid_transform<NM>(g, K, nullptr);
    for (int e = threadIdx.x; e < ntot; e += blockDim.x) {
      const int row = e / K.N1;
      const zc u = g[row * p + e - row * K.N1];
      o[e] += f * (u.x * u.x + u.y * u.y);
    }
    __syncthreads();
  }
}
__global__ void k_kpt_dens_sum(const double* __restrict__ part, int n, long ntot, double* __restrict__ dens,
                               int first) {
  for (long r = (long)blockIdx.x * blockDim.x + threadIdx.x; r < ntot; r += (long)gridDim.x * blockDim.x) {
    double s = first ? 0.0 : dens[r];
    for (int c = 0; c < n; ++c) s += part[(size_t)c * ntot + r];
    dens[r] = s;
  }
}

// ------------------------------------------------------- band products
// C[i * nb + j] = sum_g conj(A[i][g]) B[j][g], times i q_a(g) for a >= 0 (the
// derivative of a projector phase e^{-i(k+G).R}).  One wavefront per 2 x 2
// outputs; blockIdx.y: the product of the launch (S and H together), or the
// axis of the projector derivative.
__global__ void __launch_bounds__(256) k_kpt_zdot(const KptDev* __restrict__ kd, KptProduct p0, KptProduct p1) {
  const KptDev& k = kd[blockIdx.z];
  const KptProduct pr = blockIdx.y == 0 ? p0 : p1;
  const int na = pr.a == W_BETA ? k.nproj : k.nb, nb = k.nb, npw = k.npw;
  const int ti = (na + 1) / 2, tj = (nb + 1) / 2;
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= ti * tj) return;
  const int i0 = w / tj * 2, j0 = (w % tj) * 2;
  const zc* a0 = band_array(k, pr.a) + (size_t)i0 * npw;
  const zc* a1 = i0 + 1 < na ? a0 + npw : a0;
  const zc* b0 = band_array(k, pr.b) + (size_t)j0 * npw;
  const zc* b1 = j0 + 1 < nb ? b0 + npw : b0;
  zc s[4] = {};
  for (int g = lane; g < npw; g += 64) {
    const zc x0 = a0[g], x1 = a1[g], y0 = b0[g], y1 = b1[g];
    s[0] = zfma(zconj(x0), y0, s[0]);
    s[1] = zfma(zconj(x0), y1, s[1]);
    s[2] = zfma(zconj(x1), y0, s[2]);
    s[3] = zfma(zconj(x1), y1, s[3]);
  }
  zc* C = pr.out == 0 ? k.S : (pr.out == 1 ? k.H : (pr.out == 2 ? k.C : k.P));
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    s[q] = {wave_sum(s[q].x), wave_sum(s[q].y)};
    const int i = i0 + q / 2, j = j0 + q % 2;
    if (lane == 0 && i < na && j < nb) C[(size_t)i * nb + j] = s[q];
  }
}
// dP[a][p][n] = sum_g conj(beta[p][g]) i q_a(g) X[n][g] (the nonlocal forces)
__global__ void __launch_bounds__(256) k_kpt_dproj(const KptDev* __restrict__ kd) {
  const KptDev& k = kd[blockIdx.z];
  const int nb = k.nb, npw = k.npw;
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= k.nproj * nb) return;
  const int p = w / nb, n = w - p * nb;
  const zc* a = k.beta + (size_t)p * npw;
  const zc* b = k.X + (size_t)n * npw;
  const double* q = k.q;
  zc s[3] = {};
  for (int g = lane; g < npw; g += 64) {
    const zc t = zcmul(a[g], b[g]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      s[c].x -= q[3 * g + c] * t.y;
      s[c].y += q[3 * g + c] * t.x;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    s[c] = {wave_sum(s[c].x), wave_sum(s[c].y)};
    if (lane == 0) k.dP[((size_t)c * k.nproj + p) * nb + n] = s[c];
  }
}

// dst[i][g] = beta dst[i][g] + alpha sum_j s_j src[j][g] m[j][i] (s_j = h[j] when h
// is given, else 1), m = M, C or P by `mat`.  A block stages GB coefficients of
// every source row in LDS, so dst may be src (the rotation of the bands);
// blockIdx.y picks src/dst among the arrays of `which` (four bits each).
__global__ void __launch_bounds__(256) k_kpt_zgemm(const KptDev* __restrict__ kd, int src, int which, int mat,
                                                   double alpha, double beta, const double* __restrict__ h,
                                                   int GB) {
  const KptDev& k = kd[blockIdx.z];
  const int npw = k.npw, nb = k.nb;
  const int g0 = blockIdx.x * GB;
  if (g0 >= npw) return;
  const int arr = (which >> (4 * blockIdx.y)) & 15;
  zc* Y = band_array(k, arr);
  const zc* X = src < 0 ? Y : band_array(k, src);
  const int nx = src == W_BETA ? k.nproj : nb;
  const zc* m = mat == 0 ? k.M : (mat == 1 ? k.C : k.P);
  extern __shared__ __align__(16) char smem[];
  zc* xs = (zc*)smem;  // [nx][GB]
  const int ng = min(GB, npw - g0);
  for (int e = threadIdx.x; e < nx * GB; e += blockDim.x) {
    const int j = e / GB, g = e - j * GB;
    const zc v = g < ng ? X[(size_t)j * npw + g0 + g] : zc{0.0, 0.0};
    xs[e] = h ? zscale(v, h[j]) : v;
  }
  __syncthreads();
  const int g = threadIdx.x % GB, groups = blockDim.x / GB;
  for (int i = threadIdx.x / GB * 2; i < nb; i += groups * 2) {
    const bool two = i + 1 < nb;
    zc s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
#pragma unroll 4
    for (int j = 0; j < nx; ++j) {
      const zc x = xs[j * GB + g];
      s0 = zfma(x, m[(size_t)j * nb + i], s0);
      s1 = zfma(x, m[(size_t)j * nb + i + (two ? 1 : 0)], s1);
    }
    if (g >= ng) continue;
    zc* y = Y + (size_t)i * npw + g0 + g;
    if (beta == 0.0) {
      *y = zscale(s0, alpha);
      if (two) y[npw] = zscale(s1, alpha);
    } else {
      *y = {fma(alpha, s0.x, beta * y->x), fma(alpha, s0.y, beta * y->y)};
      if (two) y[npw] = {fma(alpha, s1.x, beta * y[npw].x), fma(alpha, s1.y, beta * y[npw].y)};
    }
  }
}

// ------------------------------------------------------------ projectors
// beta_{k,Ilm}(G) = p_l(|k+G|) (-i)^l Y_lm(k+G) e^{-i(k+G).R_I} / sqrt(Omega)
// with the normalised Gaussian radial projectors (l = 0, 1) of the Gamma
// setup, evaluated at q = k + G.
__global__ void k_kpt_beta(const KptDev* __restrict__ kd, const int* __restrict__ patom,
                           const int* __restrict__ plm, const double* __restrict__ pr,
                           const double* __restrict__ pos, double omega) {
  const KptDev& k = kd[blockIdx.z];
  const int p = blockIdx.y, npw = k.npw;
  const double* q = k.q;
  zc* beta = k.beta;
  const int I = patom[p], l = plm[p] >> 2, m = plm[p] & 3;
  const double rl = pr[p];
  const double pi = 3.14159265358979323846;
  const double inv = 1.0 / sqrt(omega);
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < npw; g += gridDim.x * blockDim.x) {
    const double q0 = q[3 * g], q1 = q[3 * g + 1], q2 = q[3 * g + 2];
    const double qq = sqrt(q0 * q0 + q1 * q1 + q2 * q2);
    double val;
    if (l == 0) {
      val = 4.0 * pi * sqrt(pi) * pow(rl, 1.5) * exp(-0.5 * qq * qq * rl * rl) /
            sqrt(0.5 * sqrt(pi)) * (1.0 / sqrt(4.0 * pi));
    } else {
      const double qm = m == 0 ? q0 : (m == 1 ? q1 : q2);
      val = 4.0 * pi * sqrt(pi) * pow(rl, 2.5) * exp(-0.5 * qq * qq * rl * rl) /
            sqrt(0.75 * sqrt(pi)) * sqrt(3.0 / (4.0 * pi)) * qm;
    }
    val *= inv;
    double sn, cs;
    sincos(-(q0 * pos[3 * I] + q1 * pos[3 * I + 1] + q2 * pos[3 * I + 2]), &sn, &cs);
    zc v = {val * cs, val * sn};
    if (l == 1) v = {v.y, -v.x};  // times -i
    beta[(size_t)p * npw + g] = v;
  }
}

// ------------------------------------------------- complex subspace step
//   S = L L^H (Cholesky, lower), W = L^-1, H' = W H W^H, cyclic complex
//   Jacobi H' = V diag V^H, M = W^H V with eigenvalues ascending.
// New band i = sum_j old band j M[j][i].  fail receives 1 if S is not positive
// definite (M = 1 then).
//
// The rotation of a pair (p, q), a = H'_pq: U = [[c, t], [-t*, c]] with t = s
// e^{i arg a} zeroes it for tan(2 theta) = 2 |a| / (a_qq - a_pp); as in the real
// case c^2 = (1 + |d| h) / 2, h = 1 / sqrt(d^2 + 4 |a|^2), and t = sgn(d) a h / c,
// so the phase of a never has to be taken.
__device__ __forceinline__ void zjac_rotation(double app, double aqq, zc a, double* c, zc* t) {
  double d = aqq - app;
  double a2 = fma(a.x, a.x, a.y * a.y);
  const bool on = a2 > 1e-34 * fabs(app * aqq) + 1e-300;
  double h2 = fma(d, d, 4.0 * a2);
  if (__any(h2 > 1e280)) {
    const double f = h2 > 1e280 ? 0x1p-520 : 1.0;
    d *= f;
    a = zscale(a, f);
    h2 = fma(d, d, 4.0 * fma(a.x, a.x, a.y * a.y));
  }
  const double h = rsq_nr(h2);
  const double u = fma(0.5 * fabs(d), h, 0.5);
  const double rc = rsq_nr(u);
  const double cc = u * rc, f = copysign(h * rc, d);
  const zc tt = zscale(a, f);
  const double e = 0.5 * fma(-tt.y, tt.y, fma(-tt.x, tt.x, fma(-cc, cc, 1.0)));
  *c = on ? fma(cc, e, cc) : 1.0;
  *t = on ? zc{fma(tt.x, e, tt.x), fma(tt.y, e, tt.y)} : zc{0.0, 0.0};
}
__device__ __forceinline__ zc zreadlane(zc v, int lane) { return {readlane_d(v.x, lane), readlane_d(v.y, lane)}; }
__device__ __forceinline__ zc zbperm(int at, zc v) { return {bperm_d(at, v.x), bperm_d(at, v.y)}; }
// The columns of a row vector: v_p' = c v_p - t* v_q, v_q' = t v_p + c v_q, then
// the entries move as in jac_row_step.
__device__ __forceinline__ void zjac_row_step(zc& top, zc& bot, double c, zc t, bool is0, bool is_last) {
  const zc a = {fma(c, top.x, -(t.x * bot.x + t.y * bot.y)), fma(c, top.y, -(t.x * bot.y - t.y * bot.x))};
  const zc b = {fma(c, bot.x, t.x * top.x - t.y * top.y), fma(c, bot.y, t.x * top.y + t.y * top.x)};
  const zc an = {dpp_d<kDppWaveShl1>(a.x), dpp_d<kDppWaveShl1>(a.y)};
  const zc bn = {dpp_d<kDppWaveShr1>(b.x), dpp_d<kDppWaveShr1>(b.y)};
  const zc x = {is_last ? b.x : an.x, is_last ? b.y : an.y};
  top = {is0 ? a.x : x.x, is0 ? a.y : x.y};
  bot = {is0 ? x.x : bn.x, is0 ? x.y : bn.y};
}

__device__ __forceinline__ void kpt_sub_failed(const KptDev& k, int* fail) {
  const int n = k.nb;
  if (threadIdx.x == 0) *fail = 1;
  for (int e = threadIdx.x; e < n * n; e += blockDim.x) k.M[e] = (e / n == e % n) ? zc{1.0, 0.0} : zc{0.0, 0.0};
}

// The whole step for up to 8 R bands (R = 4: 32, R = 8: 64), laid out as the
// real one (kernels_sub.hip): elimination on [S | I] with the rows in registers,
// one lower triangle of H' by position (an entry whose next position lies
// above the diagonal is stored conjugated), double-buffered, one block a lane,
// M's rows rotated by the wavefronts without blocks, a round behind.  Bound by
// the dependent chain of a round (LDS read, rotation, exchange, update, barrier),
// (n - 1) rounds a sweep: 2 k-points of 20 bands take 58.6 us together, where the
// pairs in turn, with the matrices in global memory, took 604 us each.  R = 8 keeps
// 84 bytes a lane in scratch memory (16 wavefronts leave 128 registers): a solve at
// 64 bands is 3.8 times as fast as at 65, in global memory (2 k-points, 24^3, three
// iterations: 14.8 and 55.7 ms).
template <int R>
constexpr int kpt_sub_threads() { return R == 4 ? 512 : 1024; }
template <int R>
constexpr size_t kpt_sub_lds() {
  return sizeof(zc) * (2 * (size_t)(8 * R) * (8 * R + 1) + 2 * 64) + 2 * 32 * 3 * sizeof(double);
}
template <int R>
__global__ void __launch_bounds__(kpt_sub_threads<R>()) k_kpt_sub(const KptDev* __restrict__ kd, int max_sweeps,
                                                                  int* __restrict__ fail) {
  const KptDev& kp = kd[blockIdx.x];
  constexpr int N = 8 * R, LD = N + 1, TRI = N * (N + 1) / 2;
  constexpr int STR = R == 4 ? 16 : 32, RPW = 64 / STR, SETS = R == 4 ? 2 : 5;
  const int n = kp.nb, n2 = n + (n & 1), np = n2 / 2, m = n2 - 1;
  const int tid = threadIdx.x, lane = tid & 63, W = blockDim.x >> 6;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  extern __shared__ __align__(16) char smem[];
  zc* Hl = (zc*)smem;
  zc* Wl = Hl + N * LD;
  zc* prow = Wl + N * LD;
  double* cs = (double*)(prow + 2 * 64);  // [2][32][3]: c, t of two rounds
  __shared__ double sh[16 * 2];
  __shared__ int rank[N];
  for (int u = w; u < n; u += W)
    if (lane < n) {
      const zc a = kp.H[u * n + lane], b = kp.H[lane * n + u];
      Hl[u * LD + lane] = {0.5 * (a.x + b.x), 0.5 * (a.y - b.y)};
    }
  // rows of S, then of W, as in the real step
  zc v[R];
  double dc = 1.0;  // the pivot of this lane's column
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = w + 8 * r;
    const bool in = w < 8 && i < n && lane < n;
    v[r] = in ? zc(kp.S[max(i, lane) * n + min(i, lane)]) : zc{0.0, 0.0};
    if (lane > i) v[r].y = -v[r].y;
    if (lane == i) v[r].y = 0.0;
  }
  bool ok = true;
#pragma unroll
  for (int r0 = 0; r0 < R; ++r0) {
    for (int kk = 0; kk < 8; ++kk) {
      const int k = r0 * 8 + kk;
      if (k >= n || !ok) break;
      zc* row = prow + (k & 1) * 64;
      if (w == kk) row[lane] = v[r0];
      __syncthreads();
      zc p = row[lane];
      const double d = readlane_d(p.x, k);
      if (!(d > 0.0)) {
        ok = false;
        break;
      }
      double inv = rcp_nr(d);
      inv = fma(inv, fma(-d, inv, 1.0), inv);
      if (lane == k) {
        dc = d;
        p = {0.0, 0.0};
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r < r0 || (r == r0 && w <= kk)) continue;
        const zc f = zscale(zreadlane(v[r], k), -inv);
        v[r] = zfma(f, p, v[r]);
      }
    }
  }
  if (!ok) {  // the same for every thread
    kpt_sub_failed(kp, fail);
    return;
  }
  const double dinv = -1.0 / dc;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = w + 8 * r;
    const double f = 1.0 / sqrt(readlane_d(dc, i & 63));
    v[r] = lane < i ? zscale(v[r], f * dinv) : zc{lane == i ? f : 0.0, 0.0};
    if (w < 8 && i < n && lane < n) Wl[i * LD + lane] = v[r];
  }
  __syncthreads();
  // H' = W H W^H
  zc t[R], hh[R];
#pragma unroll
  for (int r = 0; r < R; ++r) t[r] = hh[r] = {0.0, 0.0};
  if (w < 8) {
    for (int k = 0; k < n; ++k) {
      const zc x = Hl[k * LD + min(lane, N - 1)];
#pragma unroll
      for (int r = 0; r < R; ++r) t[r] = zfma(zreadlane(v[r], k), x, t[r]);
    }
    for (int k = 0; k < n; ++k) {
      const zc x = zconj(Wl[min(lane, N - 1) * LD + k]);
#pragma unroll
      for (int r = 0; r < R; ++r) hh[r] = zfma(zreadlane(t[r], k), x, hh[r]);
    }
  }
  __syncthreads();  // H is read
  zc* T = Hl;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = w + 8 * r;
    if (w < 8 && i < n && lane <= i) T[i * (i + 1) / 2 + lane] = {hh[r].x, lane == i ? 0.0 : hh[r].y};
  }
  if (n2 > n && w == 0 && lane <= n) T[n * (n + 1) / 2 + lane] = {0.0, 0.0};
  __syncthreads();
  const int nblk = np * (np + 1) / 2, NH = (nblk + 63) / 64;
  JacBlock blk;
  const bool on = w * 64 + lane < nblk;
  blk.init<false>(min(w * 64 + lane, nblk - 1), n2);
  // sign of the stored imaginary parts: entry (u, v) at its next positions
  double sg[4];
  {
    const int u[2] = {jac_next(blk.P, n2), jac_next(n2 - 1 - blk.P, n2)};
    const int x[2] = {jac_next(blk.Q, n2), jac_next(n2 - 1 - blk.Q, n2)};
#pragma unroll
    for (int q = 0; q < 4; ++q) sg[q] = u[q & 1] >= x[q >> 1] ? 1.0 : -1.0;
  }
  const int k = min(lane, np - 1);
  const int ia = jac_tri(k, k), ib = jac_tri(n2 - 1 - k, n2 - 1 - k), ic = jac_tri(n2 - 1 - k, k);
  const int pP = 4 * blk.P, pQ = 4 * blk.Q;
  const bool diag = blk.P == blk.Q;
  const int kv = lane & (STR - 1), ibot = n2 - 1 - kv;
  const bool is0 = kv == 0, is_last = kv == np - 1;
  const int wv = w - NH, Wv = W - NH, tot = (n + RPW - 1) / RPW;
  const int nsets = w >= NH && wv < tot ? (tot - wv + Wv - 1) / Wv : 0;
  zc vt[SETS], vb[SETS];
#pragma unroll
  for (int q = 0; q < SETS; ++q) {
    const int j = (wv + q * Wv) * RPW + lane / STR;
    const bool in = q < nsets && j < n && kv < np;
    vt[q] = in ? zconj(Wl[kv * LD + j]) : zc{0.0, 0.0};
    vb[q] = in && ibot < n ? zconj(Wl[ibot * LD + j]) : zc{0.0, 0.0};
  }
  int par = 0;
  bool pending = false;
  auto rows = [&](int b) {
    const double* z = cs + (b * 32 + min(kv, np - 1)) * 3;
    const double c = z[0];
    const zc tt = {z[1], z[2]};
#pragma unroll
    for (int q = 0; q < SETS; ++q)
      if (q < nsets) zjac_row_step(vt[q], vb[q], c, tt, is0, is_last);
  };
  for (int sweep = 0; sweep < (n > 1 ? max_sweeps : 0); ++sweep) {
    {
      double z[2] = {0.0, 0.0};
      for (int u = w; u < n2; u += W)
        for (int q = lane; q <= u; q += 64) {
          const zc a = T[par * TRI + u * (u + 1) / 2 + q];
          if (q == u) z[1] += a.x * a.x;
          else z[0] += a.x * a.x + a.y * a.y;
        }
      block_sum<2>(z, sh);
      if (__builtin_amdgcn_readfirstlane((int)!(2.0 * z[0] > 1e-26 * z[1] + 1e-300))) break;
    }
    for (int r = 0; r < m; ++r) {
      if (w < NH) {
        const zc* A = T + par * TRI;
        zc* B = T + (TRI - par * TRI);
        const double app = A[ia].x, aqq = A[ib].x;
        const zc aqp = A[ic];
        zc x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = A[blk.rd[q]];
        double c;
        zc tt;
        zjac_rotation(app, aqq, zconj(aqp), &c, &tt);
        const double cP = bperm_d(pP, c), cQ = bperm_d(pQ, c);
        const zc tP = zbperm(pP, tt), tQ = zbperm(pQ, tt);
        if (w == 0 && lane < np) {
          double* z = cs + (par * 32 + lane) * 3;
          z[0] = c;
          z[1] = tt.x;
          z[2] = tt.y;
        }
        const zc a11 = x[0], a21 = x[1], a12 = zconj(x[2]), a22 = zconj(x[3]);
        // rows: b1 = c a1 - t a2, b2 = t* a1 + c a2
        const zc mP = zscale(tP, -1.0), cjP = zconj(tP);
        const zc b11 = zfma(mP, a21, zscale(a11, cP)), b21 = zfma(cjP, a11, zscale(a21, cP));
        const zc b12 = zfma(mP, a22, zscale(a12, cP)), b22 = zfma(cjP, a12, zscale(a22, cP));
        // columns: r1 = c b1 - t* b2, r2 = t b1 + c b2
        const zc mQ = {-tQ.x, tQ.y};
        zc r[4] = {zfma(mQ, b12, zscale(b11, cQ)), zfma(mQ, b22, zscale(b21, cQ)),
                   zfma(tQ, b11, zscale(b12, cQ)), zfma(tQ, b21, zscale(b22, cQ))};
        if (diag) {
          r[0].y = r[3].y = 0.0;
          if (tP.x != 0.0 || tP.y != 0.0) r[1] = r[2] = {0.0, 0.0};
        }
        if (on) {
#pragma unroll
          for (int q = 0; q < 4; ++q) B[blk.wr[q]] = {r[q].x, sg[q] * r[q].y};
        }
      } else if (pending && nsets > 0) {
        rows(par ^ 1);
      }
      pending = true;
      par ^= 1;
      __syncthreads();
    }
  }
  if (pending && nsets > 0) rows(par ^ 1);
  const zc* D = T + par * TRI;
  for (int i = tid; i < n; i += blockDim.x) {
    const double li = D[jac_tri(i, i)].x;
    int rnk = 0;
    for (int j = 0; j < n; ++j) {
      const double lj = D[jac_tri(j, j)].x;
      if (lj < li || (lj == li && j < i)) ++rnk;
    }
    rank[i] = rnk;
    kp.eps[rnk] = li;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < SETS; ++q) {
    const int j = (wv + q * Wv) * RPW + lane / STR;
    if (q < nsets && j < n && kv < np) {
      kp.M[j * n + rank[kv]] = vt[q];
      if (ibot < n) kp.M[j * n + rank[ibot]] = vb[q];
    }
  }
}

// More bands: one workgroup, matrices in global memory (n x n complex,
// row-major), the rounds' disjoint pairs in parallel.
__global__ void __launch_bounds__(512) k_kpt_sub_large(const KptDev* __restrict__ kd, int max_sweeps,
                                                       int* __restrict__ fail) {
  const KptDev& kp = kd[blockIdx.x];
  const int n = kp.nb;
  zc *S = kp.S, *H = kp.H, *W = kp.W, *V = kp.V, *M = kp.M;
  double* eps = kp.eps;
  const int tid = threadIdx.x, nthr = blockDim.x;
  __shared__ int bad;
  __shared__ double sh[16 * 2];
  __shared__ int rank[320];
  __shared__ double rc[160];
  __shared__ zc rt[160];
  if (tid == 0) bad = 0;
  __syncthreads();
  // Cholesky, in place in S (lower triangle)
  for (int k = 0; k < n; ++k) {
    const double d = S[(size_t)k * n + k].x;
    if (!(d > 0.0)) {
      if (tid == 0) bad = 1;
      break;
    }
    const double piv = sqrt(d), ip = 1.0 / piv;
    __syncthreads();
    for (int i = k + 1 + tid; i < n; i += nthr) S[(size_t)i * n + k] = zscale(S[(size_t)i * n + k], ip);
    __syncthreads();
    if (tid == 0) S[(size_t)k * n + k] = {piv, 0.0};
    const int m = n - k - 1;
    for (int t = tid; t < m * m; t += nthr) {
      const int i = k + 1 + t / m, j = k + 1 + t % m;
      if (j <= i)
        S[(size_t)i * n + j] = zsub(S[(size_t)i * n + j], zmul(S[(size_t)i * n + k], zconj(S[(size_t)j * n + k])));
    }
    __syncthreads();
  }
  __syncthreads();
  if (bad) {
    kpt_sub_failed(kp, fail);
    return;
  }
  // W = L^-1 by forward substitution, one column per thread group
  for (int e = tid; e < n * n; e += nthr) W[e] = {0.0, 0.0};
  __syncthreads();
  for (int c = tid; c < n; c += nthr) {
    for (int i = c; i < n; ++i) {
      zc s = i == c ? zc{1.0, 0.0} : zc{0.0, 0.0};
      for (int k = c; k < i; ++k) s = zsub(s, zmul(S[(size_t)i * n + k], W[(size_t)k * n + c]));
      W[(size_t)i * n + c] = zscale(s, 1.0 / S[(size_t)i * n + i].x);
    }
  }
  __syncthreads();
  // H' = W H W^H: first T = W H into V, then H' = T W^H into S
  for (int e = tid; e < n * n; e += nthr) {
    const int i = e / n, j = e % n;
    zc s = {0.0, 0.0};
    for (int k = 0; k <= i; ++k) s = zadd(s, zmul(W[(size_t)i * n + k], H[(size_t)k * n + j]));
    V[e] = s;
  }
  __syncthreads();
  for (int e = tid; e < n * n; e += nthr) {
    const int i = e / n, j = e % n;
    zc s = {0.0, 0.0};
    for (int k = 0; k <= j; ++k) s = zadd(s, zmul(V[(size_t)i * n + k], zconj(W[(size_t)j * n + k])));
    S[e] = s;
  }
  __syncthreads();
  // Hermitian part, V = I
  for (int e = tid; e < n * n; e += nthr) {
    const int i = e / n, j = e % n;
    if (i < j) {
      const zc a = S[(size_t)i * n + j], b = zconj(S[(size_t)j * n + i]);
      const zc h = {0.5 * (a.x + b.x), 0.5 * (a.y + b.y)};
      S[(size_t)i * n + j] = h;
      S[(size_t)j * n + i] = zconj(h);
    } else if (i == j) {
      S[e].y = 0.0;
    }
    V[e] = i == j ? zc{1.0, 0.0} : zc{0.0, 0.0};
  }
  __syncthreads();
  // rounds of disjoint pairs (the circle schedule, by index): position u of
  // round r holds index jac_index(u, r), pair k the positions k and n2 - 1 - k
  const int n2 = n + (n & 1), np = n2 / 2, m = n2 - 1;
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    double v[2] = {0.0, 0.0};
    for (int e = tid; e < n * n; e += nthr) {
      const zc a = S[e];
      if (e / n == e % n) v[1] += a.x * a.x;
      else v[0] += a.x * a.x + a.y * a.y;
    }
    block_sum<2>(v, sh);
    if (!(v[0] > 1e-26 * v[1] + 1e-300)) break;
    for (int r = 0; r < m; ++r) {
      if ((tid & ~63) < np) {
        const int k = min(tid, np - 1), p = jac_index(k, r, m), q = jac_index(n2 - 1 - k, r, m);
        const bool in = p < n && q < n;
        const int pc = min(p, n - 1), qc = min(q, n - 1);
        double c;
        zc t;
        zjac_rotation(S[(size_t)pc * n + pc].x, S[(size_t)qc * n + qc].x,
                      in ? S[(size_t)pc * n + qc] : zc{0.0, 0.0}, &c, &t);
        if (tid < np) {
          rc[tid] = c;
          rt[tid] = t;
        }
      }
      __syncthreads();
      for (int e = tid; e < np * np + np * n; e += nthr) {
        if (e < np * np) {  // rows of pair P and columns of pair Q of H'
          const int P = e / np, Q = e - P * np;
          const int p1 = jac_index(P, r, m), p2 = jac_index(n2 - 1 - P, r, m);
          const int q1 = jac_index(Q, r, m), q2 = jac_index(n2 - 1 - Q, r, m);
          const zc z0 = {0.0, 0.0};
          const bool i1 = p1 < n, i2 = p2 < n, j1 = q1 < n, j2 = q2 < n;
          const zc a11 = i1 && j1 ? S[(size_t)p1 * n + q1] : z0, a12 = i1 && j2 ? S[(size_t)p1 * n + q2] : z0;
          const zc a21 = i2 && j1 ? S[(size_t)p2 * n + q1] : z0, a22 = i2 && j2 ? S[(size_t)p2 * n + q2] : z0;
          const double cP = rc[P], cQ = rc[Q];
          const zc tP = rt[P], tQ = rt[Q], mP = zscale(tP, -1.0), cjP = zconj(tP), mQ = {-tQ.x, tQ.y};
          const zc b11 = zfma(mP, a21, zscale(a11, cP)), b21 = zfma(cjP, a11, zscale(a21, cP));
          const zc b12 = zfma(mP, a22, zscale(a12, cP)), b22 = zfma(cjP, a12, zscale(a22, cP));
          zc r11 = zfma(mQ, b12, zscale(b11, cQ)), r21 = zfma(mQ, b22, zscale(b21, cQ));
          zc r12 = zfma(tQ, b11, zscale(b12, cQ)), r22 = zfma(tQ, b21, zscale(b22, cQ));
          if (P == Q) {
            r11.y = r22.y = 0.0;
            if (tP.x != 0.0 || tP.y != 0.0) r12 = r21 = z0;
          }
          if (i1 && j1) S[(size_t)p1 * n + q1] = r11;
          if (i1 && j2) S[(size_t)p1 * n + q2] = r12;
          if (i2 && j1) S[(size_t)p2 * n + q1] = r21;
          if (i2 && j2) S[(size_t)p2 * n + q2] = r22;
        } else {  // columns of V
          const int u = e - np * np, P = u / n, i = u - P * n;
          const int p1 = jac_index(P, r, m), p2 = jac_index(n2 - 1 - P, r, m);
          if (p1 >= n || p2 >= n) continue;
          const zc a = V[(size_t)i * n + p1], b = V[(size_t)i * n + p2], t = rt[P];
          V[(size_t)i * n + p1] = zfma(zc{-t.x, t.y}, b, zscale(a, rc[P]));
          V[(size_t)i * n + p2] = zfma(t, a, zscale(b, rc[P]));
        }
      }
      __syncthreads();
    }
  }
  // ascending order (ties by index); M = W^H V with columns by rank
  for (int i = tid; i < n; i += nthr) {
    const double li = S[(size_t)i * n + i].x;
    int r = 0;
    for (int j = 0; j < n; ++j) {
      const double lj = S[(size_t)j * n + j].x;
      if (lj < li || (lj == li && j < i)) ++r;
    }
    rank[i] = r;
  }
  __syncthreads();
  for (int e = tid; e < n * n; e += nthr) {
    const int j = e / n, i = e % n;
    zc s = {0.0, 0.0};
    for (int k = j; k < n; ++k) s = zadd(s, zcmul(W[(size_t)k * n + j], V[(size_t)k * n + i]));
    M[(size_t)j * n + rank[i]] = s;
  }
  for (int i = tid; i < n; i += nthr) eps[rank[i]] = S[(size_t)i * n + i].x;
}

// ------------------------------------------------------ CG and line search
__device__ __forceinline__ double tpa_k(double x) {
  const double p = 27.0 + x * (18.0 + x * (12.0 + 8.0 * x));
  return p / (p + 16.0 * x * x * x * x);
}

// residual R = H x - eps x, Teter-Payne-Allan preconditioned g = K R,
// D = g + (gamma / gamma_prev) D_prev (Fletcher-Reeves on the
// preconditioned norm); one workgroup per band
__global__ void __launch_bounds__(256) k_kpt_cg_dir(const KptDev* __restrict__ kd, int first) {
  const KptDev& k = kd[blockIdx.y];
  const int i = blockIdx.x, npw = k.npw;
  __shared__ double sh[16];
  const zc* x = k.X + (size_t)i * npw;
  const zc* hx = k.HX + (size_t)i * npw;
  zc* d = k.D + (size_t)i * npw;
  const double* kin = k.kin;
  double v[1] = {0.0};
  for (int g = threadIdx.x; g < npw; g += blockDim.x) v[0] += kin[g] * (x[g].x * x[g].x + x[g].y * x[g].y);
  block_sum<1>(v, sh);
  const double ek = fmax(v[0], 1e-8), e = k.eps[i];
  double w[1] = {0.0};
  for (int g = threadIdx.x; g < npw; g += blockDim.x) {
    const zc r = {hx[g].x - e * x[g].x, hx[g].y - e * x[g].y};
    w[0] += tpa_k(kin[g] / ek) * (r.x * r.x + r.y * r.y);
  }
  block_sum<1>(w, sh);
  const double gm = w[0];
  const double beta = first ? 0.0 : (k.gam[i] > 0.0 ? gm / k.gam[i] : 0.0);
  for (int g = threadIdx.x; g < npw; g += blockDim.x) {
    const double kk = tpa_k(kin[g] / ek);
    const zc r = {hx[g].x - e * x[g].x, hx[g].y - e * x[g].y};
    const zc dp = first ? zc{0.0, 0.0} : d[g];
    d[g] = {kk * r.x + beta * dp.x, kk * r.y + beta * dp.y};
  }
  __syncthreads();  // every thread has read the previous norm
  if (threadIdx.x == 0) k.gam[i] = gm;
}

// exact minimiser of the 2x2 Rayleigh quotient in span{x, d / |d|} (d is
// orthogonal to every band): theta = atan2(-2b, c - a) / 2 with
// a = <x|H|x>, b = Re<x|H|d>/|d|, c = <d|H|d>/|d|^2
__global__ void __launch_bounds__(256) k_kpt_linemin(const KptDev* __restrict__ kd) {
  const KptDev& k = kd[blockIdx.y];
  const int i = blockIdx.x, npw = k.npw;
  __shared__ double sh[16 * 4];
  zc* x = k.X + (size_t)i * npw;
  zc* hx = k.HX + (size_t)i * npw;
  const zc* d = k.D + (size_t)i * npw;
  const zc* hd = k.HD + (size_t)i * npw;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int g = threadIdx.x; g < npw; g += blockDim.x) {
    v[0] += x[g].x * hx[g].x + x[g].y * hx[g].y;
    v[1] += x[g].x * hd[g].x + x[g].y * hd[g].y;
    v[2] += d[g].x * hd[g].x + d[g].y * hd[g].y;
    v[3] += d[g].x * d[g].x + d[g].y * d[g].y;
  }
  block_sum<4>(v, sh);
  if (!(v[3] > 0.0)) return;
  const double inv = 1.0 / sqrt(v[3]);
  const double a = v[0], b = v[1] * inv, c = v[2] * inv * inv;
  const double th = 0.5 * atan2(-2.0 * b, c - a);
  double sn, cs;
  sincos(th, &sn, &cs);
  const double s2 = sn * inv;
  for (int g = threadIdx.x; g < npw; g += blockDim.x) {
    x[g] = {cs * x[g].x + s2 * d[g].x, cs * x[g].y + s2 * d[g].y};
    hx[g] = {cs * hx[g].x + s2 * hd[g].x, cs * hx[g].y + s2 * hd[g].y};
  }
}

// random starting bands, damped by 1/(1 + |k+G|^2/2) (counter-based hash of
// (seed, k, band, coefficient))
__device__ __forceinline__ double hash_unit(unsigned long long z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (double)(z >> 11) * (1.0 / 9007199254740992.0) - 0.5;
}
__global__ void k_kpt_init(const KptDev* __restrict__ kd, unsigned seed) {
  const KptDev& k = kd[blockIdx.y];
  const int npw = k.npw, kidx = blockIdx.y;
  const long n = (long)k.nb * npw;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    const int g = (int)(e % npw);
    const unsigned long long base = ((unsigned long long)seed << 40) ^ ((unsigned long long)kidx << 32) ^
                                    (unsigned long long)e * 2ull;
    const double s = 1.0 / (1.0 + k.kin[g]);
    k.X[e] = {hash_unit(base) * s, hash_unit(base + 1) * s};
  }
}

// ------------------------------------------------ occupations, density
// Occupations over every k with one chemical potential (Fermi-Dirac,
// sum_k w_k sum_n f_nk = N_el) or fixed (the lowest N_el/2 states of each k
// doubly occupied); writes occ[k][n] and the band energy, entropy and mu
// into the structure's status block (slots as at Gamma).  One workgroup; the
// bracket of mu is narrowed by one point per wavefront and round, as at Gamma
// (2 x 20 levels: 23 us; 1,665 us with one thread's bisection).
constexpr int kKptOccWaves = 16;
__global__ void __launch_bounds__(64 * kKptOccWaves) k_kpt_occupations(const double* __restrict__ eps,
                                                                       const double* __restrict__ wk, int nk,
                                                                       int nb, double nelec, int kind,
                                                                       double sigma, double* __restrict__ occ,
                                                                       double* __restrict__ scal) {
  const int n = nk * nb, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  __shared__ double sh[16 * 2];
  __shared__ double bounds[2][kKptOccWaves];
  const int nocc = (int)(nelec / 2.0 + 0.5);
  // fixed: the highest filled and the lowest empty level; else the bracket
  double lo = 1e300, hi = -1e300;
  for (int e = tid; e < n; e += blockDim.x) {
    const int i = e % nb;
    if (kind == 0) {
      occ[e] = i < nocc ? 2.0 : 0.0;
      if (i == nocc - 1) hi = fmax(hi, eps[e]);
      if (i == nocc) lo = fmin(lo, eps[e]);
    } else {
      lo = fmin(lo, eps[e]);
      hi = fmax(hi, eps[e]);
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o, 64));
    hi = fmax(hi, __shfl_xor(hi, o, 64));
  }
  if (lane == 0) {
    bounds[0][w] = lo;
    bounds[1][w] = hi;
  }
  __syncthreads();
  for (int k = 0; k < kKptOccWaves; ++k) {
    lo = fmin(lo, bounds[0][k]);
    hi = fmax(hi, bounds[1][k]);
  }
  double v[2] = {0.0, 0.0};
  double mu;
  if (kind == 0) {
    mu = nocc < nb ? 0.5 * (hi + lo) : hi;
    for (int e = tid; e < n; e += blockDim.x) v[0] += e % nb < nocc ? wk[e / nb] * 2.0 * eps[e] : 0.0;
  } else {
    lo -= 40.0 * sigma;
    hi += 40.0 * sigma;
    __shared__ int over[2][kKptOccWaves];
    const double e0 = lane < n ? eps[lane] : 0.0, w0 = lane < n ? 2.0 * wk[lane / nb] : 0.0;
    for (int it = 0; it < 80; ++it) {
      const double mid = 0.5 * (lo + hi);
      if (mid <= lo || mid >= hi) break;
      const double at = fmin(fmax(lo + (hi - lo) * ((w + 1) / (kKptOccWaves + 1.0)), lo), hi);
      double s = lane < n ? w0 / (1.0 + exp((e0 - at) / sigma)) : 0.0;
      for (int e = lane + 64; e < n; e += 64) s += wk[e / nb] * 2.0 / (1.0 + exp((eps[e] - at) / sigma));
      s = wave_sum(s);
      if (lane == 0) over[it & 1][w] = s > nelec;
      __syncthreads();
      const unsigned long long many = __ballot(lane < kKptOccWaves && over[it & 1][lane & (kKptOccWaves - 1)]);
      const int k = many ? __ffsll((long long)many) - 1 : kKptOccWaves;
      const double a = lo, d = hi - lo;
      if (k > 0) lo = fmin(fmax(a + d * (k / (kKptOccWaves + 1.0)), a), hi);
      if (k < kKptOccWaves) hi = fmin(fmax(a + d * ((k + 1) / (kKptOccWaves + 1.0)), a), hi);
    }
    mu = 0.5 * (lo + hi);
    for (int e = tid; e < n; e += blockDim.x) {
      const double f = 2.0 / (1.0 + exp((eps[e] - mu) / sigma));
      occ[e] = f;
      const double g = fmin(fmax(0.5 * f, 1e-300), 1.0), gm = fmin(fmax(1.0 - 0.5 * f, 1e-300), 1.0);
      v[0] += wk[e / nb] * f * eps[e];
      v[1] += wk[e / nb] * (g * log(g) + gm * log(gm));
    }
  }
  block_sum<2>(v, sh);
  if (tid == 0) {
    scal[S_EBAND] = v[0];
    scal[S_ENTROPY] = kind == 0 ? 0.0 : -2.0 * v[1];
    scal[S_MU] = mu;
  }
}

// kinetic energy of each band, sum_G |k+G|^2/2 |c|^2
__global__ void __launch_bounds__(256) k_kpt_band_kinetic(const KptDev* __restrict__ kd) {
  const KptDev& k = kd[blockIdx.y];
  const int i = blockIdx.x;
  __shared__ double sh[16];
  const zc* x = k.X + (size_t)i * k.npw;
  const double* kin = k.kin;
  double v[1] = {0.0};
  for (int g = threadIdx.x; g < k.npw; g += blockDim.x) v[0] += kin[g] * (x[g].x * x[g].x + x[g].y * x[g].y);
  block_sum<1>(v, sh);
  if (threadIdx.x == 0) k.bandw[i] = v[0];
}

// the structure's band arrays carry the k-weighted kinetic energy for the
// energy bookkeeping of the SCF control: occ[0] = 1, bandw[0] = sum_k w_k
// sum_n f_nk E_kin,nk, the other entries 0
__global__ void __launch_bounds__(256) k_kpt_kinetic_total(const double* __restrict__ bandw_k,
                                                           const double* __restrict__ occ_k,
                                                           const double* __restrict__ wk, int nk, int nb,
                                                           double* __restrict__ occ_s,
                                                           double* __restrict__ bandw_s, int nb_s) {
  __shared__ double sh[16];
  double t[1] = {0.0};
  for (int e = threadIdx.x; e < nk * nb; e += blockDim.x) t[0] += wk[e / nb] * occ_k[e] * bandw_k[e];
  block_sum<1>(t, sh);
  for (int i = threadIdx.x; i < nb_s; i += blockDim.x) {
    occ_s[i] = i == 0 ? 1.0 : 0.0;
    bandw_s[i] = i == 0 ? t[0] : 0.0;
  }
}

// dens[r] (+)= sum over the k of the launch of w_k sum_n f_n |u_n(r)|^2 (u
// unnormalised, Omega^-1/2 applied by the density finalisation)
__global__ void k_kpt_density(const KptDev* __restrict__ kd, int nk, const zc* __restrict__ z, long ntot,
                              double* __restrict__ dens, int first) {
  for (long r = (long)blockIdx.x * blockDim.x + threadIdx.x; r < ntot; r += (long)gridDim.x * blockDim.x) {
    double t = first ? 0.0 : dens[r];
    for (int ik = 0; ik < nk; ++ik) {
      const KptDev& k = kd[ik];
      double s = 0.0;
      for (int b = 0; b < k.nb; ++b) {
        const zc u = z[((size_t)ik * k.nb + b) * ntot + r];
        s += k.occ[b] * (u.x * u.x + u.y * u.y);
      }
      t += k.w * s;
    }
    dens[r] = t;
  }
}

// Forces: nonlocal, F_I,a = -2 sum_k w_k sum_{p on I} h_p sum_n f_n
// Re[conj(P_pn) dP_pn,a] with P = <beta|u>, dP = <-i(k+G) beta|u>, plus local
// (the partial sums [nblk][nat][3]) and Ewald.  One wavefront per atom.
__global__ void __launch_bounds__(64) k_kpt_force(const KptDev* __restrict__ kd, int nk,
                                                  const double* __restrict__ h, const int* __restrict__ patom,
                                                  const double* __restrict__ floc, int nblk,
                                                  const double* __restrict__ few, int nat,
                                                  double* __restrict__ force, double* __restrict__ fnl_part) {
  const int I = blockIdx.x, lane = threadIdx.x;
  double f[3] = {0.0, 0.0, 0.0}, l[3] = {0.0, 0.0, 0.0};
  for (int ik = 0; ik < nk; ++ik) {
    const KptDev& k = kd[ik];
    const int nb = k.nb;
    for (int p = 0; p < k.nproj; ++p) {
      if (patom[p] != I) continue;
      const double c = -2.0 * k.w * h[p];
      for (int n = lane; n < nb; n += 64) {
        const zc P = k.P[(size_t)p * nb + n];
        for (int a = 0; a < 3; ++a) {
          const zc d = k.dP[((size_t)a * k.nproj + p) * nb + n];
          f[a] += c * k.occ[n] * (P.x * d.x + P.y * d.y);
        }
      }
    }
  }
  for (int b = lane; b < nblk; b += 64)
    for (int a = 0; a < 3; ++a) l[a] += floc[((size_t)b * nat + I) * 3 + a];
  for (int a = 0; a < 3; ++a) {
    f[a] = wave_sum(f[a]);
    l[a] = wave_sum(l[a]);
    if (lane == 0) {
      fnl_part[3 * I + a] = f[a];
      force[3 * I + a] = l[a] + f[a] + few[3 * I + a];
    }
  }
}

// ---------------------------------------------------------------- launchers
static int nblocks(long n, int per = 256) {
  return (int)std::max(1L, std::min(65536L, (n + per - 1) / per));
}

static size_t kpt_grid_lds(const int N[3]) { return sizeof(zc) * (size_t)(N[0] | 1) * N[1] * N[2]; }
// Longest line class of the LDS grid path, 0 where a line or the grid does not
// fit.
int kpt_lds_class(const int N[3], size_t lds_limit) {
  const int nm = std::max(N[0], std::max(N[1], N[2]));
  if (nm > 32 || kpt_grid_lds(N) > lds_limit) return 0;
  return nm <= 16 ? 16 : (nm <= 20 ? 20 : 32);
}

// Inverse (sign +1) or forward (sign -1) 3-D transforms of nb grids
// [nb][N3][N2][N1], axis by axis.
static void kpt_fft3(hipStream_t s, zc* zk, long nb, const int N[3], const FftPlan* plans, int sign) {
  const long N1 = N[0], N2 = N[1], N3 = N[2], ntot = N1 * N2 * N3;
  // (lines, A, Bs, Cs, es, plan)
  struct Ax {
    long nlines;
    int A;
    long Bs, Cs, es;
    int ax;
  } axes[3] = {{nb * N3 * N2, 1, N1, 0, 1, 0},
               {nb * N3 * N1, (int)N1, N1 * N2, 1, N1, 1},
               {nb * N2 * N1, (int)(N1 * N2), ntot, 1, N1 * N2, 2}};
  for (const Ax& a : axes) {
    const int n = plans[a.ax].n;
    const int L = std::max(1, 512 / n);
    const size_t lds = (size_t)(L * (n | 1) + n) * sizeof(zc) + n;
    hipLaunchKernelGGL(k_kpt_lines, dim3((unsigned)((a.nlines + L - 1) / L)), dim3(256), lds, s, zk,
                       plans[a.ax], a.A, a.Bs, a.Cs, a.es, a.nlines, L, sign);
    check_launch("k_kpt_lines");
  }
}

// u(r) of every band of the k-points k0 .. k0 + kc - 1 into the grids z
static void kpt_to_grid(const KptSet& K, int k0, int kc, int src) {
  kpt_zero(K.stream, K.z, (long)kc * K.nb * K.ntot);
  hipLaunchKernelGGL(k_kpt_scatter, dim3(nblocks((long)K.nb * K.npw_max), kc), dim3(256), 0, K.stream, K.dev + k0,
                     K.z, src, K.ntot);
  check_launch("k_kpt_scatter");
  kpt_fft3(K.stream, K.z, (long)kc * K.nb, K.N, K.plans, +1);
}

void kpt_zero(hipStream_t s, zc* a, long n) {
  hipLaunchKernelGGL(k_kpt_zero, dim3(nblocks(n)), dim3(256), 0, s, a, n);
  check_launch("k_kpt_zero");
}

void kpt_hpsi(const KptSet& K, int src, int dst, const double* veff, const double* h) {
  if (K.lds_class) {
    const KGrid G{K.N[0], K.N[1], K.N[2]};
    const dim3 grid(K.nb, K.nk);
    const size_t lds = kpt_grid_lds(K.N);
    if (K.lds_class == 16)
      hipLaunchKernelGGL(k_kpt_hpsi<16>, grid, dim3(256), lds, K.stream, K.dev, G, src, dst, veff);
    else if (K.lds_class == 20)
      hipLaunchKernelGGL(k_kpt_hpsi<20>, grid, dim3(256), lds, K.stream, K.dev, G, src, dst, veff);
    else
      hipLaunchKernelGGL(k_kpt_hpsi<32>, grid, dim3(256), lds, K.stream, K.dev, G, src, dst, veff);
    check_launch("k_kpt_hpsi");
  } else {
    for (int k0 = 0; k0 < K.nk; k0 += K.kchunk) {
      const int kc = std::min(K.kchunk, K.nk - k0);
      const long nb = (long)kc * K.nb;
      kpt_to_grid(K, k0, kc, src);
      hipLaunchKernelGGL(k_kpt_vmul, dim3(nblocks(nb * K.ntot)), dim3(256), 0, K.stream, K.z, veff, (int)nb, K.ntot);
      check_launch("k_kpt_vmul");
      kpt_fft3(K.stream, K.z, nb, K.N, K.plans, -1);
      hipLaunchKernelGGL(k_kpt_gather, dim3(nblocks((long)K.nb * K.npw_max), kc), dim3(256), 0, K.stream,
                         K.dev + k0, K.z, src, dst, K.ntot);
      check_launch("k_kpt_gather");
    }
  }
  if (K.nproj > 0) {
    kpt_zdot(K, 1, {W_BETA, src, 3}, {});
    kpt_zgemm(K, W_BETA, dst, 1, 2, 1.0, 1.0, h);
  }
}

void kpt_zdot(const KptSet& K, int nprod, KptProduct p0, KptProduct p1) {
  const int na = p0.a == W_BETA ? K.nproj : K.nb;
  const long tiles = (long)((na + 1) / 2) * ((K.nb + 1) / 2);
  hipLaunchKernelGGL(k_kpt_zdot, dim3((unsigned)((tiles + 3) / 4), nprod, K.nk), dim3(256), 0, K.stream, K.dev, p0, p1);
  check_launch("k_kpt_zdot");
}

void kpt_zgemm(const KptSet& K, int src, int which, int narr, int mat, double alpha, double beta,
               const double* h) {
  const int nx = src == W_BETA ? K.nproj : K.nb;
  // Coefficients staged per block: the source rows have to fit the LDS, and a
  // rough mesh of a small cell (2 x 280 coefficients) gives only 10 blocks of 64
  // per array: 11.1 us with 64, 6.0 us with 16.
  int GB = 64;
  while (GB > 1 && ((size_t)nx * GB * sizeof(zc) > 64 * 1024 ||
                    (GB > 16 && (long)(K.npw_max + GB - 1) / GB * narr * K.nk < 256)))
    GB /= 2;
  hipLaunchKernelGGL(k_kpt_zgemm, dim3((K.npw_max + GB - 1) / GB, narr, K.nk), dim3(256),
                     (size_t)nx * GB * sizeof(zc), K.stream, K.dev, src, which, mat, alpha, beta, h, GB);
  check_launch("k_kpt_zgemm");
}

void kpt_beta(const KptSet& K, const int* patom, const int* plm, const double* pr, const double* pos,
              double omega) {
  if (K.nproj == 0) return;
  hipLaunchKernelGGL(k_kpt_beta, dim3(nblocks(K.npw_max), K.nproj, K.nk), dim3(256), 0, K.stream, K.dev, patom, plm,
                     pr, pos, omega);
  check_launch("k_kpt_beta");
}

void kpt_subspace(const KptSet& K, int* fail) {
  if (K.nb <= 32)
    hipLaunchKernelGGL(k_kpt_sub<4>, dim3(K.nk), dim3(kpt_sub_threads<4>()), kpt_sub_lds<4>(), K.stream, K.dev, 60,
                       fail);
  else if (K.nb <= kKptLdsBands)
    hipLaunchKernelGGL(k_kpt_sub<8>, dim3(K.nk), dim3(kpt_sub_threads<8>()), kpt_sub_lds<8>(), K.stream, K.dev, 60,
                       fail);
  else
    hipLaunchKernelGGL(k_kpt_sub_large, dim3(K.nk), dim3(512), 0, K.stream, K.dev, 60, fail);
  check_launch("k_kpt_sub");
}

void kpt_cg_dir(const KptSet& K, int first) {
  hipLaunchKernelGGL(k_kpt_cg_dir, dim3(K.nb, K.nk), dim3(256), 0, K.stream, K.dev, first);
  check_launch("k_kpt_cg_dir");
}

void kpt_linemin(const KptSet& K) {
  hipLaunchKernelGGL(k_kpt_linemin, dim3(K.nb, K.nk), dim3(256), 0, K.stream, K.dev);
  check_launch("k_kpt_linemin");
}

void kpt_init(const KptSet& K, unsigned seed) {
  hipLaunchKernelGGL(k_kpt_init, dim3(nblocks((long)K.nb * K.npw_max), K.nk), dim3(256), 0, K.stream, K.dev, seed);
  check_launch("k_kpt_init");
}

void kpt_occupations(hipStream_t s, const double* eps, const double* wk, int nk, int nb, double nelec,
                     int kind, double sigma, double* occ, double* scal) {
  hipLaunchKernelGGL(k_kpt_occupations, dim3(1), dim3(64 * kKptOccWaves), 0, s, eps, wk, nk, nb, nelec, kind,
                     sigma, occ, scal);
  check_launch("k_kpt_occupations");
}

void kpt_kinetic(const KptSet& K, const double* bandw_k, const double* occ_k, const double* wk, double* occ_s,
                 double* bandw_s, int nb_s) {
  hipLaunchKernelGGL(k_kpt_band_kinetic, dim3(K.nb, K.nk), dim3(256), 0, K.stream, K.dev);
  check_launch("k_kpt_band_kinetic");
  hipLaunchKernelGGL(k_kpt_kinetic_total, dim3(1), dim3(256), 0, K.stream, bandw_k, occ_k, wk, K.nk, K.nb, occ_s,
                     bandw_s, nb_s);
  check_launch("k_kpt_kinetic_total");
}

void kpt_density(const KptSet& K, double* dens) {
  if (K.lds_class) {
    const KGrid G{K.N[0], K.N[1], K.N[2]};
    const size_t lds = kpt_grid_lds(K.N);
    for (int k0 = 0; k0 < K.nk; k0 += K.kchunk) {
      const int kc = std::min(K.kchunk, K.nk - k0);
      const dim3 grid(K.nchunk, kc);
      const KptDev* kd = K.dev + k0;
      if (K.lds_class == 16)
        hipLaunchKernelGGL(k_kpt_dens_lds<16>, grid, dim3(256), lds, K.stream, kd, G, K.nchunk, K.dpart);
      else if (K.lds_class == 20)
        hipLaunchKernelGGL(k_kpt_dens_lds<20>, grid, dim3(256), lds, K.stream, kd, G, K.nchunk, K.dpart);
      else
        hipLaunchKernelGGL(k_kpt_dens_lds<32>, grid, dim3(256), lds, K.stream, kd, G, K.nchunk, K.dpart);
      check_launch("k_kpt_dens_lds");
      hipLaunchKernelGGL(k_kpt_dens_sum, dim3(nblocks(K.ntot)), dim3(256), 0, K.stream, K.dpart, kc * K.nchunk,
                         K.ntot, dens, k0 == 0 ? 1 : 0);
      check_launch("k_kpt_dens_sum");
    }
    return;
  }
  for (int k0 = 0; k0 < K.nk; k0 += K.kchunk) {
    const int kc = std::min(K.kchunk, K.nk - k0);
    kpt_to_grid(K, k0, kc, W_X);
    hipLaunchKernelGGL(k_kpt_density, dim3(nblocks(K.ntot)), dim3(256), 0, K.stream, K.dev + k0, kc, K.z, K.ntot,
                       dens, k0 == 0 ? 1 : 0);
    check_launch("k_kpt_density");
  }
}

void kpt_force(const KptSet& K, const double* h, const int* patom, const double* floc, int nblk,
               const double* few, int nat, double* force, double* fnl_part) {
  if (K.nproj > 0) {
    kpt_zdot(K, 1, {W_BETA, W_X, 3}, {});
    hipLaunchKernelGGL(k_kpt_dproj, dim3((K.nproj * K.nb + 3) / 4, 1, K.nk), dim3(256), 0, K.stream, K.dev);
    check_launch("k_kpt_dproj");
  }
  hipLaunchKernelGGL(k_kpt_force, dim3(nat), dim3(64), 0, K.stream, K.dev, K.nk, h, patom, floc, nblk, few, nat, force,
                     fnl_part);
  check_launch("k_kpt_force");
}

void configure_kpt_kernels() {
  allow_lds((const void*)k_kpt_lines);
  allow_lds((const void*)k_kpt_hpsi<16>);
  allow_lds((const void*)k_kpt_hpsi<20>);
  allow_lds((const void*)k_kpt_hpsi<32>);
  allow_lds((const void*)k_kpt_dens_lds<16>);
  allow_lds((const void*)k_kpt_dens_lds<20>);
  allow_lds((const void*)k_kpt_dens_lds<32>);
  allow_lds((const void*)k_kpt_zgemm);
  allow_lds((const void*)k_kpt_sub<4>);
  allow_lds((const void*)k_kpt_sub<8>);
}

}  // namespace sgo
