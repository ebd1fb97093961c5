// Batched line transforms in LDS, in place.
//
// N = r0 r1 (r2) with radices up to 10 whose butterflies sit in a thread's
// registers (fft_reg.hpp), so most lines up to 100 (all but 75 and 96, which take
// three) take two passes over the LDS and one buffer, where radix-2/3/4/5 passes
// between two buffers take three or four.  The results are not put in order: lds_dif
// takes natural order to digit-reversed positions, the stages backwards (dit) take
// those back to natural order, and what lies between (V_eff, the density, a
// store) looks positions up in a table of N bytes.  Lines are at an odd pitch and consecutive lanes take consecutive
// lines, so the wavefront's addresses fall into different banks in every pass.
//
// With n2 = the index within a stride and L the length left to a stage,
//   lds_dif: butterfly over r at stride L / R, then times w_L^(n2 k);
//   dit:     the stages backwards, times w_L^(n2 r), then the butterfly.
// The sign is a conjugation on the way in and out (sg = +-1).
#pragma once
#include "device.hpp"
#include "fft_reg.hpp"

namespace sgo {

#define SGO_LDS_RADICES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10)

// x / d for 0 <= x < 2^20, inv = 1.0f / d (x + 1/2 keeps the product half a unit off
// the integers, relative 2^-21, above its rounding)
__device__ __forceinline__ int line_div(int x, float inv) { return (int)(((float)x + 0.5f) * inv); }

// Lines l < nl: start l ls + (l >= lo ? gap : 0), elements es apart.
struct LdsLines {
  int nl, ls, es, lo, gap;
};

// The axis' tables, by the block's threads from `first` on (one FP64 sincos
// is the longest chain of a small block, so two axes' tables are made by
// different wavefronts and next to loads in flight):
//   tw[k] = e^{+2 pi i k / n},
//   nat[p] = index held by position p after lds_dif, or pos[k] = its inverse.
__device__ __forceinline__ int lds_natural(const FftPlan& P, int p) {
  int L = P.n, mult = 1, k = 0;
  for (int s = 0; s < P.nr; ++s) {
    L = line_div(L, 1.0f / P.r[s]);
    const int d = line_div(p, 1.0f / L);
    p -= d * L;
    k += d * mult;
    mult *= P.r[s];
  }
  return k;
}
template <typename T>
__device__ __forceinline__ void lds_tables(cplx<T>* tw, unsigned char* nat, unsigned char* pos, const FftPlan& P,
                                           int first = 0) {
  const int n = P.n;
  int k = (int)threadIdx.x - first;
  if (k < 0) k += blockDim.x;
  for (; k < n; k += blockDim.x) {
    double s, c;
    sincospi(2.0 * (double)k / (double)n, &s, &c);
    tw[k] = {(T)c, (T)s};
    const int i = lds_natural(P, k);
    if (nat) nat[k] = (unsigned char)i;
    if (pos) pos[i] = (unsigned char)k;
  }
}

template <typename T, int R>
__device__ __forceinline__ void lds_stage(cplx<T>* __restrict__ A, const LdsLines& ln, int nj, int L, int st,
                                          const cplx<T>* __restrict__ tw, int tws, bool dit, T sg) {
  const float inl = 1.0f / ln.nl, ist = 1.0f / st;
  const int stride = st * ln.es;
  for (int t = threadIdx.x; t < nj * ln.nl; t += blockDim.x) {
    const int j = line_div(t, inl), l = t - j * ln.nl;
    const int b = line_div(j, ist), n2 = j - b * st;
    cplx<T>* p = A + l * ln.ls + (l >= ln.lo ? ln.gap : 0) + (b * L + n2) * ln.es;
    cplx<T> v[R], w[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v[r] = p[r * stride];
      v[r].y *= sg;
    }
    if (dit && st > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) v[r] = cmul(v[r], tw[n2 * r * tws]);
    }
    freg::fft<T, 1, R>(v, w);
    if (!dit && st > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) w[r] = cmul(w[r], tw[n2 * r * tws]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) p[r * stride] = {w[r].x, sg * w[r].y};
  }
}

// Stages s0 <= s < s1 of the lines (backwards for dit), each ended by a barrier.
template <typename T>
__device__ __forceinline__ void lds_stages(cplx<T>* A, const LdsLines& ln, const FftPlan& P, const cplx<T>* tw,
                                           bool dit, T sg, int s0, int s1) {
  for (int q = s0; q < s1; ++q) {
    const int s = dit ? s1 - 1 - (q - s0) : q;
    int L = P.n;
    for (int i = 0; i < s; ++i) L /= P.r[i];
    const int R = P.r[s], st = L / R, nj = P.n / R, tws = P.n / L;
    switch (R) {
#define SGO_RADIX(r)                                                  \
  case r:                                                             \
    lds_stage<T, r>(A, ln, nj, L, st, tw, tws, dit, sg);              \
    break;
      SGO_LDS_RADICES(SGO_RADIX)
#undef SGO_RADIX
    }
    __syncthreads();
  }
}
template <typename T>
__device__ __forceinline__ void lds_dif(cplx<T>* A, const LdsLines& ln, const FftPlan& P, const cplx<T>* tw, T sg) {
  lds_stages<T>(A, ln, P, tw, false, sg, 0, P.nr);
}

}  // namespace sgo
