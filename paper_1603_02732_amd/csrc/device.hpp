// Device helpers: wavefront/block/grid reductions, packed coefficients and the
// local-density functional.
#pragma once
#include "common.hpp"

namespace sgo {

// ---------------------------------------------------------------- reductions
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sum 64 values over the wavefront, the total of value l left in lane l: each
// step halves the values a lane holds, 63 exchanges instead of 64 x 6.
template <int O>
__device__ __forceinline__ void wave_fold(double (&v)[64]) {
  const bool up = (threadIdx.x & O) != 0;
#pragma unroll
  for (int j = 0; j < O; ++j) {
    const double keep = up ? v[j + O] : v[j], send = up ? v[j] : v[j + O];
    v[j] = keep + __shfl_xor(send, O, 64);
  }
}
__device__ __forceinline__ double wave_sum64(double (&v)[64]) {
  wave_fold<32>(v);
  wave_fold<16>(v);
  wave_fold<8>(v);
  wave_fold<4>(v);
  wave_fold<2>(v);
  wave_fold<1>(v);
  return v[0];
}

// Sum N values over the block; every thread receives the totals.  The order
// of additions is fixed by the thread layout, so results are reproducible.
// sh must hold 16*N doubles.
template <int N>
__device__ __forceinline__ void block_sum(double (&v)[N], double* sh) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = wave_sum(v[i]);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) sh[i * 16 + w] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double s = 0.0;
    for (int k = 0; k < nw; ++k) s += sh[i * 16 + k];
    v[i] = s;
  }
  __syncthreads();
}

// v[0..5] += w * (G G^T) in Voigt order xx yy zz yz xz xy.
__device__ __forceinline__ void add_voigt(double* v, double w, const double* G) {
  v[0] += w * G[0] * G[0];
  v[1] += w * G[1] * G[1];
  v[2] += w * G[2] * G[2];
  v[3] += w * G[1] * G[2];
  v[4] += w * G[0] * G[2];
  v[5] += w * G[0] * G[1];
}

__device__ __forceinline__ double load_coherent(const double* p) {
  unsigned long long u =
      __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                        __HIP_MEMORY_SCOPE_AGENT);
  return __longlong_as_double((long long)u);
}

// Grid-wide sum of N values per block.  Each block passes its block totals
// (valid in every thread); the last block to arrive sums the partials in
// block order and returns true with the totals in out (all its threads).
// The ticket is returned to zero by that block, ready for the next launch.
template <int N>
__device__ bool grid_sum_last(const double (&v)[N], double* part, unsigned* ticket, int nblocks,
                              int bid, double (&out)[N], double* sh) {
  __shared__ int is_last;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) part[(size_t)bid * N + i] = v[i];
    __threadfence();
    unsigned t = atomicAdd(ticket, 1u);
    is_last = (t == (unsigned)(nblocks - 1));
  }
  __syncthreads();
  if (!is_last) return false;
  __threadfence();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double s = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) s += part[(size_t)b * N + i];
    out[i] = s;
  }
  block_sum<N>(out, sh);
  if (threadIdx.x == 0) atomicExch(ticket, 0u);
  return true;
}

// Unpack Gamma-point storage of half-sphere coefficient g of a band:
// c_G = (x[2g] + i x[2g+1]) / sqrt2 for G != 0, c_0 = x[0].
template <typename T>
__device__ __forceinline__ cplx<T> unpack_coef(const T* x, int g) {
  const T r = (T)0.70710678118654752440;
  if (g == 0) return {x[0], (T)0};
  return {x[2 * g] * r, x[2 * g + 1] * r};
}

// Perdew-Zunger 1981 LDA (unpolarised): eps_xc and v_xc = d(rho eps)/d rho.
// The r_s >= 1 branch is taken at r_s = 1; rho <= 1e-30 gives zero.
__device__ __forceinline__ void pz81(double rho, double* eps, double* v) {
  if (!(rho > 1e-30)) {
    *eps = 0.0;
    *v = 0.0;
    return;
  }
  const double pi = 3.14159265358979323846;
  const double rs = cbrt(3.0 / (4.0 * pi * rho));
  const double ex = -0.75 * cbrt(3.0 / pi) * cbrt(rho);
  double ec, vc;
  if (rs >= 1.0) {
    const double g = -0.1423, b1 = 1.0529, b2 = 0.3334;
    const double sq = sqrt(rs);
    const double den = 1.0 + b1 * sq + b2 * rs;
    ec = g / den;
    vc = ec * (1.0 + 7.0 / 6.0 * b1 * sq + 4.0 / 3.0 * b2 * rs) / den;
  } else {
    const double A = 0.0311, B = -0.048, C = 0.0020, D = -0.0116;
    const double l = log(rs);
    ec = A * l + B + C * rs * l + D * rs;
    vc = A * l + (B - A / 3.0) + 2.0 / 3.0 * C * rs * l + (2.0 * D - C) / 3.0 * rs;
  }
  *eps = ex + ec;
  *v = 4.0 / 3.0 * ex + vc;
}

}  // namespace sgo
