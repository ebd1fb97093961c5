// Host-side launch wrappers of the HIP kernels (defined in kernels_*.hip).
#pragma once
#include "common.hpp"

namespace sgo {

// Which wavefunction-side array a kernel reads or writes.
enum WArr { W_X = 0, W_HX = 1, W_D = 2, W_HD = 3, W_BETA = 4 };
// Which FP64 matrix a product writes or reads.
enum MArr { M_S = 0, M_H = 1, M_M = 2, M_C = 3 };

// Launch geometry shared by all candidates of a batch (maxima over them).
// Default band count from which the subspace products and Jacobi rounds run
// over the whole GPU instead of one workgroup per candidate (BatchGeom
// jac_grid, tuning key SGO_JAC_GRID): one above what the one-workgroup rounds
// hold.  At 164 bands a round over the GPU is one 3.6 us launch, in one
// workgroup 1.7 us.
constexpr int kJacGridBandsDefault = 199;

// The subspace solver's part of a candidate's reduction scratch (doubles;
// free while the subspace problem is solved): the sweeps done, the ranks of
// the eigenvalues, and the rotations (c, s) of every round, for at most
// kJacMaxSweeps sweeps.
constexpr int kJacWideMax = 198;  // largest problem of the one-workgroup rounds
constexpr int kJacMaxSweeps = 40;
constexpr int kJacDone = 0;    // over the GPU: 1.0 once the candidate's H' is diagonal
constexpr int kJacSweeps = 1;
constexpr int kJacRanks = 2;   // int [640]
constexpr int kJacLog = kJacRanks + 320;
constexpr size_t jac_log_doubles(int n, int sweeps) {
  return kJacLog + (size_t)sweeps * (n + (n & 1) - 1) * (n + (n & 1));
}

struct BatchGeom {
  int ncand;
  int npair_max, nsp_max, nb_max, nproj_max, nat_max;
  int N1max, N2max, N3max, ntot_max, plane_max;
  int plane_reg;   // 1: FP32 register-FFT plane kernels for every candidate
  int pl_sx_max;   // largest compact plane row stride
  int gemm_f32;    // 1: FP32-MFMA band products in the FP32 path
  int gemm_waves = 8;  // wavefronts sharing a staged slice from 64 input rows (4, 6 or 8)
  int gram_tile = 0;   // Gram output tile: 64 rows when set to 64, else 32
  int gram_f32;    // 1: FP32-MFMA Gram products (FP64 sums of the K ranges)
  int bf16proj;    // 1: projector products with BF16 inputs (FP32_BF16PROJ form)
  size_t red_min_bytes;  // smallest reduction scratch of any candidate
  size_t lds_limit;      // dynamic LDS a kernel may use (device limit minus static use)
  int K_max;
  int sp_chunk;      // stick pairs per block of the z kernels
  int kc_len;        // K range per block of the split-K products
  int nkc_max;       // number of K ranges
  int dens_chunks;   // band-pair chunks of the density planes
  int ew_ng_max;     // reciprocal Ewald vectors enumerated (box size)
  int phase_max;         // phase factors of one candidate
  int setup_max;         // threads of the grid setup
  int nagroup_max, force_blocks_max;  // local forces: atom groups, blocks per group
  int sub_threads;   // threads of the LDS-resident subspace solver
  int jac_grid = kJacGridBandsDefault;  // band count from which the subspace solve runs over the GPU
  int plane_group = 1;  // z-planes per workgroup of the H psi plane kernel (1: one per wavefront)
};

struct LaunchCtx {
  hipStream_t stream;
  const CandDesc* desc;      // device array [ncand]
  const SpeciesDev* species; // device array [kMaxSpecies]
  BatchGeom g;
  int* jac_done = nullptr;       // device [ncand]: per-candidate Jacobi convergence flags
  int* jac_done_host = nullptr;  // pinned host copy of them
};

// False while the calling thread captures a graph (no host synchronisation).
bool host_sync_allowed();

template <typename T> void launch_hpsi(const LaunchCtx& L, int src /*W_X or W_D*/);
template <typename T> void launch_density(const LaunchCtx& L);
template <typename T> void launch_gram(const LaunchCtx& L, int nprod, const int* a, const int* b,
                                       const int* out);
template <typename T> void launch_gemm_acc(const LaunchCtx& L, int narr, const int* y, const int* a,
                                           int mat, double alpha, double beta, int use_h);
template <typename T> void launch_cg_direction(const LaunchCtx& L, int first);
template <typename T> void launch_linemin(const LaunchCtx& L);
template <typename T> void launch_band_kinetic(const LaunchCtx& L);
template <typename T> void launch_init_random(const LaunchCtx& L);
template <typename T> void launch_setup_beta(const LaunchCtx& L);
template <typename T> void launch_force_nonlocal(const LaunchCtx& L);
template <typename T> void launch_stress_waves(const LaunchCtx& L);
template <typename T> void launch_potential_finalize(const LaunchCtx& L);
void launch_subspace(const LaunchCtx& L, int mode, int max_sweeps = kJacMaxSweeps);
// Its parts: the one-workgroup step up to kJacWideMax bands (kernels_sub.hip; at
// most kJacMaxSweeps sweeps, whatever is asked for) and the products that it
// shares with the larger problems.
void launch_sub_block(hipStream_t st, const CandDesc* desc, int ncand, int n, int mode, int max_sweeps);
void launch_sub_congruence(hipStream_t st, const CandDesc* desc, int ncand, int n);
void configure_sub_kernels();
// The subspace step with its workspace in a fixed per-device array (no
// allocation): S, H (mode 3) device inputs [n*n], M [n*n] and eps [n] device
// outputs; n <= kNoAllocMaxN.  With status != NULL it only enqueues on
// `stream` and a kernel writes 0 or fail_code to *status; otherwise it waits
// for the stream and returns 0 or fail_code.
constexpr int kNoAllocMaxN = 256;
int subspace_noalloc(int device, int n, int mode, const double* S, const double* H, double* M,
                     double* eps, int* status, int fail_code, hipStream_t stream, int nthreads);
void launch_occupations(const LaunchCtx& L);
void launch_grid_fft(const LaunchCtx& L, int sign);
void launch_density_finalize(const LaunchCtx& L);
void launch_gspace_residual(const LaunchCtx& L);
// res_tol > 0: convergence also needs the charged bands' residuals at the
// gate (max(res_tol, 0.1 sqrt(tol_e_atom))).
void launch_scf_control(const LaunchCtx& L, double tol_e_atom, double tol_rho, double res_tol);
// Residual gate of the CG steps (masks candidates whose bands meet the
// residual condition, device side) and its release (phase 0, then 1).
void launch_cg_gate(const LaunchCtx& L, double tol);
// Converged or failed candidates masked on the device (multi-iteration graphs).
void launch_mask_done(const LaunchCtx& L);
void launch_cg_release(const LaunchCtx& L, int phase);
void launch_iter_set(const LaunchCtx& L, int* state, int value, int add);
void launch_mix(const LaunchCtx& L, int initial, double alpha, double q0);
void launch_setup_grid(const LaunchCtx& L);
void launch_ewald(const LaunchCtx& L);
void launch_force_local(const LaunchCtx& L);
void launch_force_finalize(const LaunchCtx& L);
void launch_stress_grid(const LaunchCtx& L);
void launch_gather_scal(const LaunchCtx& L, double* out);  // [ncand][S_COUNT]  // grid, Ewald and finalize kernels
// positions of every candidate from pos [all atoms][3], status scalars to zero
void launch_scatter_state(const LaunchCtx& L, const double* pos);
// total energies [ncand], then forces [all atoms][3]
void launch_gather_results(const LaunchCtx& L, double* out);

// Enable large dynamic LDS for every kernel (once per process per device).
void configure_kernels();
// Register-FFT plane kernels (FP32, line lengths 2^a 3^b 5^c up to 64).
bool plane_reg_length_ok(int n);
size_t plane_reg_lds(const BatchGeom& g, bool density);
void launch_plane_hpsi_reg(const LaunchCtx& L);
// Planes per workgroup of the grouped H psi plane kernel for this geometry
// (1: the one-plane kernel; `forced` > 0 asks for that size where it fits).
int plane_group_size(const BatchGeom& g, size_t lds_per_cu, int forced);
size_t plane_group_lds(const BatchGeom& g, int group);
void launch_plane_density_reg(const LaunchCtx& L);
void launch_z_inverse_reg(const LaunchCtx& L, int src);
void launch_z_forward_reg(const LaunchCtx& L, int src, int dst);
void configure_plane_kernels();
// ---- k-point sampling (kernels_kpt.hip): complex bands on the shifted
// sphere |k+G|^2/2 <= Ecut of one k-point, FP64
// Device descriptor of one k-point.
struct KptDev {
  int npw, nb, nproj, pad;
  double w;                  // weight
  GPtr<const int> box;       // [npw] index of each coefficient in the [N3][N2][N1] grid
  GPtr<const double> kin;    // [npw] |k+G|^2 / 2
  GPtr<const double> q;      // [npw][3] k + G (Cartesian, bohr^-1)
  GPtr<cplx<double>> beta;   // [nproj][npw] projectors at k + G
  GPtr<cplx<double>> X;      // bands [nb][npw], H X, directions, H D
  GPtr<cplx<double>> HX;
  GPtr<cplx<double>> D;
  GPtr<cplx<double>> HD;
  GPtr<cplx<double>> S;      // [nb][nb] subspace matrices
  GPtr<cplx<double>> H;
  GPtr<cplx<double>> W;      // above kKptLdsBands
  GPtr<cplx<double>> V;
  GPtr<cplx<double>> M;
  GPtr<cplx<double>> C;
  GPtr<cplx<double>> P;      // [nproj][nb] projections, [3][nproj][nb] their derivatives
  GPtr<cplx<double>> dP;
  GPtr<double> eps;          // [nb]
  GPtr<double> occ;
  GPtr<double> gam;
  GPtr<double> bandw;
};
// All k-points of a structure: every launch covers them.
struct KptSet {
  hipStream_t stream;
  const KptDev* dev;         // device array [nk]
  int nk, nb, nproj, npw_max;
  int N[3];
  long ntot;
  const FftPlan* plans;
  int lds_class;             // kpt_lds_class of the grid
  cplx<double>* z;           // [kchunk][nb][ntot] grids (lds_class 0)
  int kchunk;                // k-points at a time: grids, or density parts
  double* dpart;             // [kchunk][nchunk][ntot] density parts (lds_class > 0)
  int nchunk;
};
// k-points whose grids (of `bytes` each) are held at a time, at least one: 256 MB
// of them fill the chip and stay in its last cache.  32 k-points of 24 bands on
// 48^3: 114 ms for three iterations with 6 at a time, 129 ms with all (1.36 GB).
inline int kpt_grid_chunk(int nk, size_t bytes) {
  const size_t c = (size_t)256000000 / (bytes ? bytes : 1);
  return c < 1 ? 1 : (c < (size_t)nk ? (int)c : nk);
}
// The largest of want, want / 2, ... 1 for which alloc(size(chunk)) succeeds; 0 if
// none does.
template <class Size, class Alloc>
int largest_chunk(int want, Size size, Alloc alloc) {
  for (int c = want;; c = (c + 1) / 2) {
    if (alloc(size(c))) return c;
    if (c == 1) return 0;
  }
}
// conj(a) . b into matrix out: 0 S, 1 H, 2 C, 3 P (a = W_BETA)
struct KptProduct {
  int a, b, out;
};
constexpr int kKptLdsBands = 64;  // subspace matrices in LDS up to here, above in W and V
int kpt_lds_class(const int N[3], size_t lds_limit);
void kpt_zero(hipStream_t s, cplx<double>* a, long n);
void kpt_hpsi(const KptSet& K, int src, int dst, const double* veff, const double* h);
void kpt_zdot(const KptSet& K, int nprod, KptProduct p0, KptProduct p1);
// dst <- beta dst + alpha src . mat (0 M, 1 C, 2 P) for the narr arrays `which`
// (four bits each); src < 0: the array itself
void kpt_zgemm(const KptSet& K, int src, int which, int narr, int mat, double alpha, double beta,
               const double* h);
void kpt_beta(const KptSet& K, const int* patom, const int* plm, const double* pr, const double* pos,
              double omega);
void kpt_subspace(const KptSet& K, int* fail);
void kpt_cg_dir(const KptSet& K, int first);
void kpt_linemin(const KptSet& K);
void kpt_init(const KptSet& K, unsigned seed);
void kpt_occupations(hipStream_t s, const double* eps, const double* wk, int nk, int nb, double nelec,
                     int kind, double sigma, double* occ, double* scal);
void kpt_kinetic(const KptSet& K, const double* bandw_k, const double* occ_k, const double* wk, double* occ_s,
                 double* bandw_s, int nb_s);
void kpt_density(const KptSet& K, double* dens);
void kpt_force(const KptSet& K, const double* h, const int* patom, const double* floc, int nblk,
               const double* few, int nat, double* force, double* fnl_part);
void configure_kpt_kernels();
// BF16-input projector products (FP32_BF16PROJ form).
void launch_beta_bf16(const LaunchCtx& L);
void launch_proj_bf16(const LaunchCtx& L, int src, int dst);
// Raise the dynamic-LDS limit of one kernel to what the device allows.
void allow_lds(const void* kernel);
// Report a failed launch by kernel name (throws on the host side).
void check_launch(const char* name);
// Throws the library error for a failed HIP runtime call.
void hip_check(hipError_t e, const char* what);
// Reject a launch shape the kernels do not support (throws on the host side).
void throw_unsupported(const char* what);
// Optional event timing of every launch of one named kernel.
void prof_before(const char* name, hipStream_t s);
// `rows`: coefficient rows (band or projector rows of length K) that one
// candidate's share of the launch reads or writes, where a launcher states it
void prof_after(const char* name, hipStream_t s, long long rows = 0);

}  // namespace sgo
