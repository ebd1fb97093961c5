// Shared device/host definitions of the HIP engine.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sgo {

template <typename T>
struct cplx {
  T x, y;
};

template <typename T>
__device__ __forceinline__ cplx<T> cmul(cplx<T> a, cplx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ __forceinline__ cplx<T> cmulc(cplx<T> a, cplx<T> b) {  // a * conj(b)
  return {a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y};
}
template <typename T>
__device__ __forceinline__ cplx<T> cadd(cplx<T> a, cplx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ cplx<T> csub(cplx<T> a, cplx<T> b) { return {a.x - b.x, a.y - b.y}; }

constexpr int kMaxFftN = 128;     // longest 1-D transform along any axis
constexpr int kMaxHist = 8;       // Pulay history slots
constexpr int kNT = 256;          // threads of most kernels

// Scalars kept per candidate in device memory (double slots).
enum Scal {
  S_ETOT = 0, S_EKIN, S_ENL, S_ELOC, S_EH, S_EXC, S_EEW, S_ENTROPY_TERM,
  S_EBAND, S_VRHO, S_DRHO, S_DE, S_EPREV, S_MU, S_ENTROPY, S_CONV,
  S_ERR, S_ITER, S_NHIST, S_NSCF, S_EHARRIS, S_EWRECIP,
  S_CGSKIP, S_CGHOLD,  // residual gate of the CG steps (set and cleared within an iteration)
  S_COUNT = 32
};

// Radix plan of one transform length.
struct FftPlan {
  int n;     // line length
  int nr;    // stages of the in-place LDS transform (fft_lds.hpp)
  int r[3];  // their radices, descending
};

// Pointer of the descriptor: on the device it is a pointer to global memory
// (converted where it is used), so the accesses compile to global loads and
// stores.  As a plain pointer read from memory it could point into LDS as far
// as the compiler knows: every access was a flat one, which also waits on the
// LDS counter and which no later load may overtake.
#ifdef __HIP_DEVICE_COMPILE__
template <typename T>
struct GPtr {
  __attribute__((address_space(1))) T* p;
  __device__ __forceinline__ operator T*() const { return (T*)p; }
  template <typename U>  // of the untyped ones
  __device__ __forceinline__ explicit operator U*() const {
    return (U*)(T*)p;
  }
  GPtr() = default;
  __host__ __device__ GPtr(T* q) : p((__attribute__((address_space(1))) T*)q) {}
};
#else
template <typename T>
using GPtr = T*;
#endif

// Per-candidate device descriptor.  Pointers typed void* hold arrays of the
// wavefunction precision T (float or double); double* arrays are FP64.
struct CandDesc {
  int N1, N2, N3, ntot;
  int npwh, K, nb, npair;
  int Kp, pad_kp;   // Kp: row stride of band arrays (K rounded up to 32, zero padded)
  int nsp, nst, nproj, nat;
  int occ_kind, nocc, active, ncand_index;
  int pl_nx, pl_nxl, pl_sx;  // active x columns of the planes (register FFT kernels)
  int pos_off;               // start of this candidate in arrays [all atoms][3]
  int np16, pad_np;     // nproj rounded up to 16 (BF16 projector tiles)
  double sigma, nelec, omega, pad0;
  double A[9];
  double B[9];
  FftPlan plan[3];  // lengths N1, N2, N3
  // wavefunction side (precision T)
  GPtr<void> X;
  GPtr<void> HX;
  GPtr<void> D;
  GPtr<void> HD;
  GPtr<void> sticks;   // cplx<T> [npair][N3][nst]
  GPtr<void> veff_t;   // T [N3][N2][N1]
  GPtr<void> beta;     // T [nproj][K]
  GPtr<void> beta16;   // bfloat16 [2][np16][Kp] hi, lo parts (FP32_BF16PROJ form only)
  GPtr<void> betaT16;  // bfloat16 [2][Kp][np16]
  GPtr<const double> kin;     // [npwh]
  GPtr<const int> gmeta;      // [npwh] stick | z << 20
  GPtr<const int> sp_off;     // [nsp + 1]
  GPtr<const int> stick_xy;   // [nst] i1 | i2 << 16
  GPtr<const int> gmill;      // [npwh*3] Miller indices of the half sphere
  GPtr<const double> hproj;   // [nproj]
  GPtr<const int> proj_atom;  // [nproj]
  GPtr<const int> proj_lm;    // [nproj] l*4 + m
  GPtr<const double> proj_r;  // [nproj] projector width
  // subspace (FP64)
  GPtr<double> S;       // [nb*nb]
  GPtr<double> Hs;      // [nb*nb]
  GPtr<double> M;       // [nb*nb]
  GPtr<double> C;       // [max(nb,nproj)*nb] general product
  GPtr<double> eps;     // [nb]
  GPtr<double> occ;     // [nb]
  GPtr<double> gam;     // [nb]  gamma of the previous CG step
  GPtr<double> bandw;   // [nb]  per-band scratch
  GPtr<double> resn;    // [nb]  |H psi - eps psi|^2 of each band at the last CG direction
  // grid side (FP64)
  GPtr<double> rho_in_r;     // [ntot]
  GPtr<double> rho_out_r;    // [ntot]
  GPtr<double> veff_r;       // [ntot]
  GPtr<cplx<double>> zgrid;  // [ntot] FFT work
  GPtr<cplx<double>> vloc_G; // [ntot] on D, zero elsewhere
  GPtr<cplx<double>> rho0_G; // [ntot]
  GPtr<cplx<double>> rho_out_G;  // [ntot]
  GPtr<void> hist_in;            // [kMaxHist][ntot] complex, FP64 or FP32 (hist_f32)
  GPtr<void> hist_res;           // [kMaxHist][ntot]
  GPtr<double> pulay;        // [kMaxHist*kMaxHist] residual dot products
  GPtr<double> coef;         // [kMaxHist]
  GPtr<double> dens_part;    // [nchunk][ntot]
  int ndens_chunk;
  int hist_len;         // history capacity in use
  int hist_f32;         // Pulay history stored as complex FP32 (FP32 bulk forms)
  // atoms (FP64)
  GPtr<const double> pos;    // [nat*3]
  GPtr<const int> spec;      // [nat]
  // phase factors e^{i m b_a.R_I}, m >= 0: phase[(I * 3 + a) * phase_m + m]
  GPtr<cplx<double>> phase;
  int phase_m;          // entries per atom and axis: max(N_a / 2, ew_m[a]) + 1
  int nagroup;          // atom groups: at most kAtomGroup atoms of one species
  GPtr<const int> agroup;    // [nagroup * kAtomGroup] atom indices, -1 past a group's end
  GPtr<double> force;        // [nat*3] total
  GPtr<double> force_ew;     // [nat*3]
  GPtr<double> force_part;   // [nat*3*4] local / nonlocal scratch
  GPtr<double> nlwork;       // [nproj*nb*4]
  GPtr<double> stwork;       // stress partial sums, layout in stress_layout()
  GPtr<double> stress;       // [9] total, then [6][9] parts (kin, nl, H, loc, xc, Ewald)
  GPtr<double> scal;         // [S_COUNT]
  GPtr<cplx<double>> ewS;    // [ew_ng] Ewald structure factors
  double ew_eta, ew_rcut, ew_gcut, pad2;
  int ew_m[3], ew_n[3];  // reciprocal / image enumeration half-widths
  int ew_ng, ew_nimg;
  GPtr<long long> dbg_clk;   // optional phase timestamps of the subspace solver
  GPtr<int> iter_state;      // SCF iteration counter of the batch (device memory)
  // reduction scratch: partial sums and tickets (zeroed at allocation)
  GPtr<double> red_part;     // [kRedSlots]
  GPtr<unsigned> tickets;    // [kTickets]
  unsigned seed;
  int pad1;
};

constexpr int kRedSlots = 1 << 16;

// Local forces: a block sums kNT columns of the half grid (m1 >= 0) over
// kForceZ planes for one atom group; their partial sums, [block][nat][3], lie
// in red_part.
constexpr int kAtomGroup = 8;
constexpr int kForceZ = 16;
constexpr int kSetupZ = 4;  // planes a thread of the geometry setup takes
__host__ __device__ inline int force_blocks(int N1, int N2, int N3) {
  return ((N1 + 1) / 2 * N2 + kNT - 1) / kNT * ((N3 + kForceZ - 1) / kForceZ);
}

// Stress partial sums (doubles): per band kinetic [nb][6]; per projector and
// band (P, Q_xx..Q_xy) [nproj][nb][7]; grid blocks [kStressBlocks][16];
// per atom Ewald [nat][13].  Voigt order xx yy zz yz xz xy.
constexpr int kStressBlocks = 256;
struct StressLayout {
  size_t kin, nl, grid, ew, total;
};
__host__ __device__ inline StressLayout stress_layout(int nb, int nproj, int nat) {
  StressLayout L;
  L.kin = 0;
  L.nl = (size_t)6 * nb;
  L.grid = L.nl + (size_t)7 * nproj * nb;
  L.ew = L.grid + (size_t)16 * kStressBlocks;
  L.total = L.ew + (size_t)13 * nat;
  return L;
}
constexpr int kTickets = 512;
constexpr int kTicketGrid = 480;  // first ticket not used by the Gram products

// Species parameters on device (constant per batch).
struct SpeciesDev {
  double Z;
  int local_kind;
  int nkb;
  double p[3];
  int kb_l[4];
  double kb_r[4];
  double kb_h[4];
  double rho0_width;
};
constexpr int kMaxSpecies = 16;

}  // namespace sgo
