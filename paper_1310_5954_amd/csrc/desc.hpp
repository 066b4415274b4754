// Device-resident descriptors shared by the runtime and the kernels.
//
// An instance is one resident AO filter (its ensemble, D, domain map and
// scratch live in one workspace).  A batch is a list of instances that have
// one frame each in the current launch sequence; kernels are launched once
// per (padded ensemble size, storage precision) class and walk the class's
// entries, so the frames of several instances share every launch.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace letkf {

constexpr int kMaxBatch = 64;   // frames per batch
constexpr int kParkDoubles = 128 * 112;  // 64 < m <= 128, poly: a parking slot (isqrt_stages)
constexpr int kParkSlots = 256; // most workgroups of such an analysis launch, and parking slots of an instance
// classes 0..15: 4 padded sizes (16, 32, 64, 128) x 4 arithmetic variants
// (index variant x 4 + size): FP64, FP32, BF16, and BF16 with the Jacobi
// rotations in FP32 (LETKF_FLAG_FP32_ROTATIONS); class 16: 129..256 members,
// FP64 only
constexpr int kVariants = 4;
constexpr int kNumClasses = 4 * kVariants + 1;
constexpr int kBigClass = 4 * kVariants;

struct InstState {           // mutated on the device by the forecast kernel
  int32_t cur;               // ring slot holding phi_k (the other holds phi_{k-1})
  int32_t unconverged;       // domains of the last analysis that hit the Jacobi sweep cap or whose stages did not get there
  uint64_t frame;            // forecasts done so far (Philox counter word 2..3)
  unsigned long long sweeps; // Jacobi sweeps (poly: matrix products of the stages) summed over every domain solve
  unsigned long long solves; // domain solves
};

struct InstDesc {
  int32_t n_act, n_sub, m, n_dom;
  int32_t prec, flags, zrows, nnz;
  int32_t obs_inst;          // ring slot offset of the observed instant: 0 = phi_k, 1 = phi_{k-1}
  int32_t poly;              // 1: k_analysis_poly analyses the instance, 0: k_analysis (uses_poly)
  double sigma_v;
  double a_diag;             // (m-1)/rho
  double sqrt_m1;            // (m-1)^(1/2)
  uint64_t seed;
  void* ens;                 // [2][n_act][m]   storage type (double for FP64, float otherwise)
  void* Yp;                  // [p][m]          slope perturbations D X'_phi
  double* d;                 // [p]             innovation y - D xbar_phi
  void* Z;                   // [zrows][m]      per-domain analysis rows before the merge
  const double* a1;          // [n_act]
  const double* a2;          // [n_act]
  const int32_t* d_rowptr;   // [p+1]
  const int32_t* d_col;      // [nnz]
  const double* d_val;       // [nnz]
  const int32_t* dom;        // [n_dom][4]: est_off, e, obs_off, s  (Z rows of l start at 2*est_off)
  const int32_t* order;      // [n_dom] domains by decreasing estimated cost
  const int32_t* est_act;    // [sum e]
  const int32_t* obs_row;    // [2 sum s]: slope row of each observation (x rows then y rows per domain)
  const double* obs_r;       // [2 sum s]: taper * R^-1 of each observation (null where no kernel reads it: reads_weights)
  const double* obs_sr;      // [2 sum s]: its square root (the weight of the staged rows of C)
  const int32_t* mptr;       // [n_act+1] merge CSR: covering (domain, position) entries per actuator
  const int32_t* mrow;       // [2*entries]: Z row of the phi_k copy and of the phi_{k-1} copy
  const double* mw;          // [entries]: merge weight
  const int32_t* mdom;       // [entries]: domain of each merge entry
  const double* pist_op;     // [n_dom][n_dom] piston operator (NULL unless LETKF_FLAG_PISTONS)
  const int32_t* pist_ptr;   // [n_dom+1] CSR of each domain's mismatch terms
  const int32_t* pist_row;   // [2*terms]: Z row of the term at phi_k and at phi_{k-1}
  const double* pist_coef;   // [terms]: its coefficient (1, or 1 - k_j for the domain's own row)
  double* pist_r;            // [n_dom][2][m] overlap mismatch of each domain, instant, member
  double* pist_c;            // [n_dom][2][m] pistons added before the merge
  double* bigA;              // m > 128: [n_dom][256][256] A
  double* bigW;              // m > 128: [n_dom][5][256][256] M, M^2, P and two Z of the stages (column-major)
  double* bigv;              // m > 128: [n_dom][5][256] b, wbar, shift and exponent, partial sums of norms, the stages' plan
  const uint8_t* guess;      // poly: [n_dom] first entry of the stages (stage_guess)
  int32_t* bigf;             // m > 128: [n_dom][4] debug Jacobi: converged, rounds that rotated, sweeps; stages done
  uint32_t* dom_sweeps;      // [n_dom] Jacobi sweeps (poly: products) of each domain, summed over every analysis
  double* Ascr;              // FP64, m <= 128: [n_dom][m(m+1)/2] each domain's A (lower triangle packed by rows), for refining wbar
  double* park;              // poly, 64 < m <= 128: [min(n_dom, kParkSlots)][kParkDoubles] a workgroup's Z between its stages
  double* dbg;               // [n_dom][2*m*m + m] C, lambda, T (NULL unless debug)
  int32_t* dbg_sweeps;       // [n_dom]
  InstState* st;
};

// Entries of one class in a batch.  Prefix arrays index the flattened work of
// the class: actuator rows, slope rows and domains of every entry.
struct ClassBatch {
  int32_t n;
  int32_t inst[kMaxBatch];        // index into the instance table
  int32_t ent[kMaxBatch];         // batch entry (position of y / outputs)
  int32_t act_off[kMaxBatch + 1];
  int32_t slope_off[kMaxBatch + 1];
  int32_t dom_off[kMaxBatch + 1];
  uint32_t next;                  // analysis work counter: items claimed past the first grid (k_slopes zeroes it)
  uint32_t next_poly;             // the same for k_analysis_poly
};

struct BatchHdr {
  const double* yptr[kMaxBatch];  // slopes of entry e (device memory: staging slot or caller's buffer)
  double* amean;                  // analysis means (phi_k), entry e at out_off[e]
  double* pmean;                  // prediction means (phi_{k+1}), entry e at out_off[e]
  int32_t out_off[kMaxBatch];
  // check_y != 0 (server batches): the slope kernel sets bad[e] when entry e's
  // slopes hold a non-finite value, and the merge/forecast kernels then leave
  // that instance's ensemble and frame counter as they were.  The host uploads
  // the header with bad[] zeroed for every batch.
  int32_t check_y;
  int32_t bad[kMaxBatch];
  ClassBatch cls[kNumClasses];
};

// Per-domain debug record (LETKF_FLAG_DEBUG): C [m*m], lambda [m], T [m*m],
// then kDbgTail slots: 0-5 shader-clock stamps at the 6 phase boundaries,
// 6 HW_ID, 7 XCC_ID, 8 the workgroup index that ran the domain, 10-12 stamps
// inside the wbar/W/T phase (after U, after wbar, after its refinement).
constexpr int kDbgTail = 16;

// Arithmetic variant of an instance: its precision path, or 3 for the BF16
// path with FP32 rotations (fp32_rot: LETKF_FLAG_FP32_ROTATIONS, validated to
// come with LETKF_BF16).
inline int variant_of(int prec, bool fp32_rot) { return fp32_rot ? 3 : prec; }

// Which analysis kernel serves an instance (m <= 128): A^(-1/2) by polynomial
// stages (k_analysis_poly) or through the Jacobi eigensolver (k_analysis).  The
// stages are as accurate as the eigensolver on X' W (isqrt_stages) and take 0.47
// of its launch time in FP64 at 84 x 84, m = 64 (135 against 286 us), so they
// serve every instance whose trajectory a change of rounding leaves alone.
// Three kinds do not.  The
// BF16 paths round X' to BF16 every frame, so that two solvers agreeing to 1e-7
// flip different roundings and stand 1e-3 apart after four to eight frames.  On
// the FP32 path the rounding of C and of the state, amplified by kappa(A) and by
// the filter, does the same at a smaller scale: 3e-7 to 1e-5 after 16 frames on
// most maps with m <= 64, but up to 1e-4 with few slopes per domain or hard
// window edges, 4e-5 after two frames for m > 64, and by instance the error
// against 64 bits moves by half either way.  A filter that observes the previous
// instant (H = [0 D]) is unstable on window maps (a CPU replay of 33 x 33 grows a
// perturbation 7 times a frame).  Those keep the solver, and so the
// trajectories, they have had.
inline bool uses_poly(int prec, int obs_instant) { return prec == 0 && obs_instant == 0; }
constexpr int kKindJacobi = 1, kKindPoly = 2;  // kinds of instances in a launch

// Whether a kernel reads the observations' weights themselves and not only their
// square roots: the FP64 gathers of m > 64, but for k_analysis_poly's.
inline bool reads_weights(int prec, int padded_m, int obs_instant) {
  return prec == 0 && (padded_m > 128 || (padded_m == 128 && !uses_poly(prec, obs_instant)));
}

// Entry of the polynomial stages (kappa <= 2^(entry / 4)) for what A's condition
// number may be off the vector of ones, from the domain's observation weights r
// and the number of actuators that its slopes touch.  With n slopes against m - 1
// directions the smallest eigenvalue of C off the ones goes as
// (1 - sqrt((m-1) / n))^2 (the lower edge of a sample covariance); with fewer
// slopes than directions nothing better than the bound of (m-1)/rho is to be had
// (the last entry stands for that).  Slopes of small weight count too, at that
// weight (taken at 1, 1/8, 1/64 and 1/512 of the largest, fractions below).  The
// actuators touched, less one (piston), bound the rank in the same way.  The
// factors 96 and 16 are what the slopes' own spectrum adds: their quotient was
// 30 to 100 over the von Karman domains of 8 to 128 subapertures, 20 to 60 in
// the frames after the first.  A guess only (a certificate decides when the
// stages end), but one within a factor 10 of the truth keeps the rounding to
// that condition number's, below that of Cholesky + SVD, where the bound's
// stages cost one to three digits.
constexpr int kStageEntries = 208;
inline int stage_guess(int m, const double* r, int count, int touched) {
  auto edge = [&](double n) {  // 0: no more than the directions
    const double u = 1.0 - std::sqrt((m - 1) / n);
    return n > m - 1 ? u * u : 0.0;
  };
  double most = 0.0, kappa = HUGE_VAL, scale = 1.0;
  for (int q = 0; q < count; ++q) most = std::fmax(most, r[q]);
  for (int k = 0; k < 4 && most > 0.0; ++k, scale *= 8.0) {
    double n = 0.0;
    for (int q = 0; q < count; ++q) n += std::fmin(r[q] / most * scale, 1.0);
    kappa = std::fmin(kappa, 96.0 * scale / edge(n));
  }
  kappa = std::fmax(kappa, 16.0 / edge(touched - 1));
  return (int)std::fmin(kStageEntries, std::ceil(4.0 * std::log2(kappa)));
}

inline int class_of(int padded_m, int prec, bool fp32_rot) {
  if (padded_m > 128) return kBigClass;  // validated to be FP64
  int s = padded_m <= 16 ? 0 : padded_m <= 32 ? 1 : padded_m <= 64 ? 2 : 3;
  return variant_of(prec, fp32_rot) * 4 + s;
}

// Entries of the packed lower triangle of an n x n matrix (row i starts at tri_size(i)).
__host__ __device__ inline int tri_size(int n) { return n * (n + 1) / 2; }

inline int padded_members(int m) {
  int p = 16;
  while (p < m) p *= 2;
  return p;
}

}  // namespace letkf
