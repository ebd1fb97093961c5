// Cyclic Jacobi rounds on a symmetric FP64 matrix held in LDS by position.
//
// The round-robin (circle) schedule pairs, in every round, position k with
// position n2 - 1 - k (k < np = n2 / 2, n2 = n rounded up to even; an odd n
// gets a zero row, which no rotation touches).  Position 0 keeps its index;
// after a round the contents of positions 1 .. n2 - 1 move down by one,
// cyclically, so after the m = n2 - 1 rounds of a sweep every index is back at
// the position of its own number.  With H' stored by position (lower
// triangle, packed) a thread handles the same 2x2 blocks at the same
// addresses in every round: the loop has no index arithmetic and no pair
// lookup, and only one triangle is updated.
#pragma once
#include "device.hpp"
#include "launch.hpp"

namespace sgo {

// Addresses of the entry (u, v) = (v, u) among n2 (n2 + 1) / 2.
__device__ __forceinline__ int jac_tri(int u, int v) {  // packed lower triangle
  const int a = u > v ? u : v, b = u > v ? v : u;
  return a * (a + 1) / 2 + b;
}
// By pairs: with P >= Q the pairs that hold u and v, the block number t = P (P +
// 1) / 2 + Q within one of four triangles, (top P, top Q), (bottom P, top Q),
// (bottom P, bottom Q) and (top P, bottom Q) without P = Q.  A wavefront handles
// consecutive blocks, so its four reads are four runs of consecutive words, and
// its writes as well but for the ends of a row; packed by (u, v) half of them are
// strides of about n2, different from lane to lane.
__device__ __forceinline__ int jac_quad(int u, int v, int n2) {
  const int np = n2 / 2, M = np * (np + 1) / 2;
  const bool bu = u >= np, bv = v >= np;
  const int pu = bu ? n2 - 1 - u : u, pv = bv ? n2 - 1 - v : v;
  const bool sw = pu < pv;
  const int P = sw ? pv : pu, Q = sw ? pu : pv, t = P * (P + 1) / 2 + Q;
  const bool bP = sw ? bv : bu, bQ = sw ? bu : bv;
  if (bP == bQ) return bP ? 2 * M + t : t;
  return bP || P == Q ? M + t : 3 * M + t - P;
}
// QUAD from 65 bands on: the rounds of 112 bands 449 -> 437 us, of 164 bands 1.19 ->
// 1.00 ms a call of the engine (4 to 5 sweeps on average); up to 64 a round is a chain of latencies and the longer way to the addresses
// costs more (32 bands: 104 -> 106 us).
template <bool QUAD>
__device__ __forceinline__ int jac_addr(int u, int v, int n2) {
  return QUAD ? jac_quad(u, v, n2) : jac_tri(u, v);
}
// Where a round's results go: the contents of position u move to jac_next(u).
__device__ __forceinline__ int jac_next(int u, int n2) { return u == 0 ? 0 : (u == 1 ? n2 - 1 : u - 1); }
// Index held by position u in round r.
__device__ __forceinline__ int jac_index(int u, int r, int m) {
  if (u == 0) return 0;
  const int a = u - 1 + r;
  return (a >= m ? a - m : a) + 1;
}

// 1/x and 1/sqrt(x) from the hardware approximations refined by one Newton
// step (about 1 ulp; the rotation only has to be orthogonal to rounding).
__device__ __forceinline__ double rcp_nr(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double rsq_nr(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  return r * fma(-0.5 * x * r, r, 1.5);
}

// Rotation (c, s) that zeroes a_pq of [[app, apq], [apq, aqq]], |angle| <= 45
// degrees: tan(2 angle) = 2 apq / (aqq - app).  From the hypotenuse: with
// d = aqq - app, b = 2 apq, h = 1 / sqrt(d^2 + b^2):
//   c^2 = (1 + |d| h) / 2,  s = sgn(d) b h / (2 c),
// two reciprocal square roots in the dependent chain where the quotient form
// theta = d / b, t = 1 / (|theta| + sqrt(theta^2 + 1)) has two quotients
// besides; then (c, s) is brought to unit length (first order: its error is
// at rounding level).  Entries at rounding level (|apq| <= 1e-17
// sqrt|app aqq|) are left alone.  At d = 0 the lower index leads (`top`,
// `bot`, round r of m: the positions' indices).  Every lane of the wavefront
// takes part.
__device__ __forceinline__ void jac_rotation(double app, double aqq, double apq, int top, int bot, int r,
                                             int m, double* c, double* s) {
  double d = aqq - app, b = apq + apq;
  double h2 = fma(d, d, b * b);
  if (__any(h2 > 1e280)) {  // far from any physical H'; keeps d^2 in range
    const double f = h2 > 1e280 ? 0x1p-520 : 1.0;
    d *= f;
    b *= f;
    h2 = fma(d, d, b * b);
  }
  if (__any(d == 0.0)) {
    const bool first = jac_index(top, r, m) < jac_index(bot, r, m);
    if (d == 0.0) d = first == (b >= 0.0) ? 1e-300 : -1e-300;  // the sign alone matters
  }
  const double h = rsq_nr(h2);
  const double u = fma(0.5 * fabs(d), h, 0.5);
  const double sb = copysign(0.5, d) * b * h;
  const double rc = rsq_nr(u);
  const double cc = u * rc, ss = sb * rc;
  const double e = 0.5 * fma(-ss, ss, fma(-cc, cc, 1.0));
  const bool on = apq * apq > 1e-34 * fabs(app * aqq) + 1e-300;
  *c = on ? fma(cc, e, cc) : 1.0;
  *s = on ? fma(ss, e, ss) : 0.0;
}

__device__ __forceinline__ double readlane_d(double x, int lane) {
  const long long v = __double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(v & 0xffffffffll), lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Value of the lane with byte index `at` (4 x lane).
__device__ __forceinline__ double bperm_d(int at, double x) {
  const long long v = __double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute(at, (int)(v & 0xffffffffll));
  const unsigned hi = (unsigned)__builtin_amdgcn_ds_bpermute(at, (int)(v >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Lane i receives lane i + 1's (wave_shl) or lane i - 1's (wave_shr) value.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  const long long v = __double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(v & 0xffffffffll), CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int kDppWaveShl1 = 0x130, kDppWaveShr1 = 0x138;

// The columns of a row vector that a round's rotations act on: lane k holds
// the entries of pair k (top: position k, bot: position n2 - 1 - k).  After
// the rotations the entries move to their next positions: tops one lane
// down, bots one lane up, the last bot becomes the last top and the second
// top the first bot; top 0 stays.
__device__ __forceinline__ void jac_row_step(double& top, double& bot, double c, double s, bool is0,
                                             bool is_last) {
  const double t = fma(c, top, -(s * bot)), b = fma(s, top, c * bot);
  const double tn = dpp_d<kDppWaveShl1>(t), bn = dpp_d<kDppWaveShr1>(b);
  const double x = is_last ? b : tn;  // a single pair keeps both entries
  top = is0 ? t : x;
  bot = is0 ? x : bn;
}

// Off-diagonal norm below 1e-13 of the diagonal norm (one wavefront a row at a
// time; every thread of the block takes part).
template <bool QUAD>
__device__ __forceinline__ bool jac_converged(const double* T, int n2, double* sh) {
  const int w = threadIdx.x >> 6, W = blockDim.x >> 6, lane = threadIdx.x & 63;
  const int np = n2 / 2, M = np * (np + 1) / 2;
  double v[2] = {0.0, 0.0};
  if (QUAD) {
    for (int P = w; P < np; P += W)
      for (int Q = lane; Q <= P; Q += 64) {
        const int t = P * (P + 1) / 2 + Q;
        const double a = T[t], b = T[2 * M + t], c = T[M + t], d = P != Q ? T[3 * M + t - P] : 0.0;
        if (P == Q) v[1] += a * a + b * b;
        else v[0] += a * a + b * b + d * d;
        v[0] += c * c;
      }
  } else {
    for (int u = w; u < n2; u += W)
      for (int q = lane; q <= u; q += 64) {
        const double a = T[u * (u + 1) / 2 + q];
        if (q == u) v[1] += a * a;
        else v[0] += a * a;
      }
  }
  block_sum<2>(v, sh);
  return __builtin_amdgcn_readfirstlane((int)!(2.0 * v[0] > 1e-26 * v[1] + 1e-300)) != 0;
}

// Addresses of block t of the block triangle (P >= Q, t = P (P + 1) / 2 + Q):
// entries (top P, top Q), (bot P, top Q), (top P, bot Q), (bot P, bot Q), where a
// round reads them (rd) and where it leaves them (wr).
struct JacBlock {
  int P, Q, rd[4], wr[4];
  template <bool QUAD>
  __device__ __forceinline__ void init(int t, int n2) {
    P = (int)((sqrtf(8.0f * t + 1.0f) - 1.0f) * 0.5f);
    while (P * (P + 1) / 2 > t) --P;
    while ((P + 1) * (P + 2) / 2 <= t) ++P;
    Q = t - P * (P + 1) / 2;
    const int bp = n2 - 1 - P, bq = n2 - 1 - Q;
    const int tpn = jac_next(P, n2), bpn = jac_next(bp, n2), tqn = jac_next(Q, n2), bqn = jac_next(bq, n2);
    rd[0] = jac_addr<QUAD>(P, Q, n2);
    rd[1] = jac_addr<QUAD>(bp, Q, n2);
    rd[2] = jac_addr<QUAD>(P, bq, n2);
    rd[3] = jac_addr<QUAD>(bp, bq, n2);
    wr[0] = jac_addr<QUAD>(tpn, tqn, n2);
    wr[1] = jac_addr<QUAD>(bpn, tqn, n2);
    wr[2] = jac_addr<QUAD>(tpn, bqn, n2);
    wr[3] = jac_addr<QUAD>(bpn, bqn, n2);
  }
};
// x: the entries in that order, rotated in place; the rotated entry of a
// diagonal block itself (zeroed) is zero.
__device__ __forceinline__ void jac_block_update(double (&x)[4], double cP, double sP, double cQ, double sQ,
                                                 bool diag) {
  const double b11 = fma(cP, x[0], -(sP * x[1])), b21 = fma(sP, x[0], cP * x[1]);
  const double b12 = fma(cP, x[2], -(sP * x[3])), b22 = fma(sP, x[2], cP * x[3]);
  const double r12 = fma(sQ, b11, cQ * b12), r21 = fma(cQ, b21, -(sQ * b22));
  const bool zeroed = diag && sP != 0.0;
  x[0] = fma(cQ, b11, -(sQ * b12));
  x[1] = zeroed ? 0.0 : r21;
  x[2] = zeroed ? 0.0 : r12;
  x[3] = fma(sQ, b21, cQ * b22);
}

}  // namespace sgo
