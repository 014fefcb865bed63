// Device data layout and kernel launchers of the HEVI step (gfx950).
//
// Every field is stored [col][lev] with the levels of one column contiguous.
// Interface fields (W) use the same layout: slot j holds interface j
// (0 = ground, always 0); the lid value (j = L) is 0 and not stored.
// Launch geometry: see n_blocks (lanes = levels, cpw columns per wavefront)
// and n_blocks_h (kHq levels per lane, hcpw columns per wavefront).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "../../include/thor.h"
#include "internal.h"

namespace thor {

// Values per column of the stencil records, padded so that a record is a
// multiple of 16 bytes in either precision (they are copied in 16-byte pieces).
constexpr int kDc = 24, kLc = 8, kFr = 12, kDv = 16, kGt = 12, kDw = 2 * kRing2;

// H: horizontal-field storage/arithmetic type: double (FP64 path) or float
// (mixed-precision form).  Vertical solve, reference state and prognostic
// density / rho-theta / W stay double in both.
template <typename H>
struct Fields {
  // geometry (per column; a pentagon's missing neighbour, and a missing
  // two-ring column, is the column itself with zero weight)
  const int32_t *nbr;     // [N][6]
  const H *dc;            // [N][kDc] divergence/gradient coefficient vectors (7 x 3)
  const H *lc;            // [N][kLc] Laplacian neighbour weights (6)
  const H *rhat;          // [N][3]
  const H *frame;         // [N][kFr] local east e, north n and rhat of the column (9)
  const double *frame64;  // [N][6] e and n of the column in FP64 (mixed form only)
  const double *wind64;   // [N][6] the same of the position as the mixed form holds it (mixed form only)
  const H *dv;            // [N][kDv] divergence coefficients of (Ma, Mb): c_j . (e, n) of column j (14)
  const H *gt;            // [N][kGt] gradient coefficients in the column's own basis (6 x 2)
  const int32_t *ddi;     // [N][18] two-ring columns
  const H *ddw;           // [N][kDw] lap(grad .) weights in the column's own basis (18 x 2)
  const double *area;     // [N]
  const double *teq;      // [N] Newtonian T_eq; cos(lon - lon_ss) cos(lat) (hot Jupiter); sin(lat) (Held-Suarez)

  // current small-step state.  Inside a stage rho holds the deviation from
  // rho[t] (the stage's last substep leaves the density itself) and the
  // horizontal momentum its east and north components (Ma, Mb); the last
  // substep of a large step also leaves it as the Cartesian (Mx, My, Mz) that
  // every other reader of the state uses
  double *rho, *rth, *W;  // [N][L]
  H *Mx, *My, *Mz;        // [N][L]
  H *Ma, *Mb;             // [N][L]
  H *ps;                  // p* = p - p[t]
  // large-step copies Phi[t]
  double *rho_t, *rth_t, *W_t, *p_t;
  H *Mx_t, *My_t, *Mz_t;
  // large-step forcing (frozen over the step)
  H *FMa, *FMb;           // -grad p[t] + hyperdiffusion of momentum, tangent components
  double *FW;             // [t] vertical imbalance + hyperdiffusion of W
  H *Hrho, *Hrth;         // hyperdiffusion of rho and rho theta (horizontal stencils)
  // stage forcing
  H *SMa, *SMb;
  double *SW;
  H *thL, *Gam;           // linearisation theta and gamma p / rho theta
  // divergence damping
  H *D;                   // 3D divergence of the small-step state
  H *Dt;                  // and of Phi[t]
  // large-step temporaries
  double *wI;             // w at the interfaces (W / rho_I) of Phi[t]
  double *Xrho, *Xvx, *Xvy, *Xvz, *Xw, *XT;
  // diagnostics
  double *diag;           // [N][L]
  double *partial;        // per-block partial sums
  double *epart;          // energy fixer: partial sums of the step's start and of
                          // the dynamics output, then the temperature increment
  // anelastic switch only (null otherwise): the reference column rho_r [S]
  // (padding levels repeat the top level) and, frozen per large step,
  // rho_r / rho[t] at the centres and the ratio of the two-point means at
  // interface slot j (slot 0, the ground, holds 1)
  const double *rref;
  H *fC;                  // [N][L]
  double *fI;             // [N][L]
};

// Kernels dominated by horizontal gathers (acoustic phase M, slow terms) use
// a second mapping: each lane owns kHq consecutive levels of one column,
// hlpc = ceil(L / kHq) lanes per column and hcpw = floor(64 / hlpc) columns
// per wavefront.  Per-column stencil weights are then loaded once per kHq
// cells, rows move in 16-byte loads, and a vertical neighbour is a register
// or, across a lane boundary, one shuffle.
constexpr int kHq = 4;

// 1 / x from the hardware reciprocal estimate refined by Newton steps (two in
// FP64, one in FP32), and x / y from r = 1 / y with the remainder's correction.
// For normal operands and quotients (densities, pressures, radii, pivots).
// Nothing here proves correct rounding, but of 5.2e9 random operands in each
// precision (exponents -20 to 20) both gave the correctly rounded value every time.
// The compiler's division also scales its operands and repairs special
// cases, 11 instructions to 5 and 3: 21 of them made up 40 % of the FP64
// instructions of the slow terms, 32 were 55 % of the large step's first
// pass.  Large step g5 L37 37.2 -> 35.1 us, mixed 36.0 -> 33.1; slow terms
// 12.85 -> 12.6 and 10.1 -> 9.4; phase V 14.7 -> 14.4 and 11.7 -> 11.5.
__device__ __forceinline__ double rcpd(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}
__device__ __forceinline__ float rcpd(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}
__device__ __forceinline__ double quot(double x, double y, double r) {
  const double q = x * r;
  return fma(fma(-y, q, x), r, q);
}
__device__ __forceinline__ float quot(float x, float y, float r) {
  const float q = x * r;
  return fmaf(fmaf(-y, q, x), r, q);
}

// The kHq levels of a lane in 16-byte loads (rows have whole groups of kHq).
__device__ __forceinline__ void row4(const double *p, double v[kHq]) {
  const double2 a = *reinterpret_cast<const double2 *>(p), b = *reinterpret_cast<const double2 *>(p + 2);
  v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ __forceinline__ void row4(const float *p, float v[kHq]) {
  const float4 a = *reinterpret_cast<const float4 *>(p);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
}

// Local east and north of a column in FP64 (a mixed state's `frame` is FP32):
// tangent64 for the change of basis at the ends of a large step, of the column
// itself, as the coefficients of the step are; wind64 for what reads the winds
// of a state or corrects them (diagnostics, zonal means, network inputs,
// corrections), in the mixed form of the FP32 position.  The rounding of a
// position's z moves that north out of the column's tangent plane by up to
// 3e-8 / cos(lat), 9.7e-7 at g6, which a component along it feels in second
// order, but a momentum built from it in first: the step's own basis leaves M
// within FP32 rounding (4.4e-8 |M| at g6) of the plane.
template <typename H>
__device__ __forceinline__ void basis64(const Fields<H> &f, const double *mixed, int col, double e[3], double n[3]) {
  const double *t = sizeof(H) == sizeof(double) ? reinterpret_cast<const double *>(f.frame) + (size_t)col * kFr
                                                : mixed + (size_t)col * 6;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    e[k] = t[k];
    n[k] = t[3 + k];
  }
}
template <typename H>
__device__ __forceinline__ void tangent64(const Fields<H> &f, int col, double e[3], double n[3]) {
  basis64(f, f.frame64, col, e, n);
}
template <typename H>
__device__ __forceinline__ void wind64(const Fields<H> &f, int col, double e[3], double n[3]) {
  basis64(f, f.wind64, col, e, n);
}

struct Consts {
  int N, L, cpw;          // columns, levels, columns per wavefront
  int S;                  // row stride of the per-cell state arrays (L rounded up to a multiple of 4)
  int hlpc, hcpw;         // phase-M mapping: lanes per column, columns per wavefront
  double radius, omega, grav, Rd, Cp, Cv, gamma, p_ref;
  double dz, Kd;
  double idz, rd_p;       // 1 / dz and Rd / p_ref
  double rdz;             // radial spacing of the levels: dz, or 0 (shallow atmosphere)
  double dt;
  int div_damp;
  int energy_fixer;       // 1: uniform internal-energy fixer after the dynamics
  int hydrostatic;        // 1: no vertical acceleration in the acoustic substeps
  int shallow;            // 1: shallow atmosphere (r = radius), traditional Coriolis
  int vorder;             // order of the vertical Lagrange interpolation (1 or 3)
  int anelastic;          // 1: reference-density mass flux (needs vorder 1 and vnl 4)
  int vnl, vlpc, vcpw;    // phase V: levels per lane (1 or 2); with 2, lanes per column and columns per wavefront
  int forcing;
  double tau;
  // hot-Jupiter benchmark forcing (Eqs. teq-hj, btrop, tvert)
  double hj_Tsurf, hj_dTep, hj_lapse, hj_zstrat, hj_dTstrat, hj_sstrat;
  // Held-Suarez forcing (Eqs. im_eq_v, im_eq_fv; Sec. 7.1 T_eq, K_T)
  double hs_kf, hs_ka, hs_ks, hs_sb, hs_dTy, hs_dthz, hs_pstar, hs_Ttop, hs_Tmin;
};

// Workgroups have 1, 2, 4 or 8 wavefronts (tuned per kernel family).
constexpr int kMaxBlock = 512;
constexpr int kXcds = 8;   // MI355X: 8 accelerator complex dies, one L2 each

// Launched workgroups of `wpb` wavefronts (a multiple of kXcds; surplus
// workgroups store nothing).
inline int n_blocks_for(long n_col, int cols_per_wave, int wpb) {
  long waves = (n_col + cols_per_wave - 1) / cols_per_wave;
  long wg = (waves + wpb - 1) / wpb;
  return (int)((wg + kXcds - 1) / kXcds * kXcds);
}
inline int n_blocks(const Consts &c, int wpb) { return n_blocks_for(c.N, c.cpw, wpb); }

inline int n_blocks_h(const Consts &c, int wpb) { return n_blocks_for(c.N, c.hcpw, wpb); }
inline long n_waves_h(const Consts &c) { return (c.N + c.hcpw - 1) / c.hcpw; }

// Wavefronts of at most kLdsCols columns (13 levels and up) stage stencil
// weights in LDS, in slices of whole KiB (one copy instruction of the wavefront
// each).  A chosen limit: 8 slices of 16 columns fit a workgroup's 64 KiB in
// either precision (56 in FP64); 21 columns (9 to 12 levels) would fill it and
// 32 (5 to 8) exceed it in FP64.  Where they would fit, they pay on large grids
// only: a large step at L = 12 with them and without, g4 167 / 160 us, g5 205.5 /
// 200.5, g6 438 / 449, g7 1796 / 1986; L = 8, g6 362 / 376, g7 1202 / 1336.
constexpr int kLdsCols = 16;
__host__ __device__ inline int wave_bytes(int bytes) { return (bytes + 1023) / 1024 * 1024; }
// Per wavefront of `cols` columns in phase M (damping and gradient weights);
// 0: not staged.
template <typename H>
inline int hmom_lds(int cols) {
  return cols <= kLdsCols ? wave_bytes(cols * kDw * (int)sizeof(H)) + wave_bytes(cols * kGt * (int)sizeof(H)) : 0;
}

// In the slow terms (divergence coefficients, frame) and the large-step
// kernels (coefficients and Laplacian weights; weights, gradient, frame): g6
// L32 FP64 slow terms 40.7 -> 39.6 us, large step 112 -> 105, g7 L48 246 ->
// 238 and 641 -> 620, mixed slow terms 27.6 -> 26.6.  k_large1 stages in FP64
// only: in the mixed form, where its fields are double and its weights half
// as long, 89.1 us per large step without and 90.8 with.  Phase V's 14
// coefficients are not staged: 35.3 -> 34.8 us at g6 L32, but mixed 25.7 ->
// 26.2, g7 L48 231 -> 233.5, g4 L20 6.0 -> 6.7.
template <typename H>
constexpr bool kStageLarge1 = sizeof(H) == sizeof(double);
template <typename H>
inline int slow_lds(int cols) {
  return cols <= kLdsCols ? wave_bytes(cols * kDc * (int)sizeof(H)) + wave_bytes(cols * kFr * (int)sizeof(H)) : 0;
}
template <typename H>
inline int large1_lds(int cols) {
  return kStageLarge1<H> && cols <= kLdsCols ? wave_bytes(cols * kDc * (int)sizeof(H)) + wave_bytes(cols * kLc * (int)sizeof(H)) : 0;
}
template <typename H>
inline int large2_lds(int cols) {
  return cols <= kLdsCols ? wave_bytes(cols * kLc * (int)sizeof(H)) + wave_bytes(cols * kGt * (int)sizeof(H)) +
                                wave_bytes(cols * kFr * (int)sizeof(H))
                          : 0;
}

// Launchers.  `wpb` = wavefronts per workgroup (tuned per kernel family).
// The prognostic state between large steps lives in the *_t buffers; a large
// step reads them as Phi[t] and leaves its result in the unsuffixed buffers,
// after which the host swaps the two buffer sets.
// Acoustic substeps take dtau = dt / div (div = 3 in stage 1, n otherwise);
// first = first substep of an RK stage (restart from Phi[t], p* = 0);
// stage_end = its last one (phase V leaves the density, not its deviation);
// last = final substep of the large step (phase M then also leaves the
// Cartesian momentum; phase V applies the physics, unless the energy fixer
// does it afterwards).
// ev0 / ev1 (timing, may be null): events recorded by the dispatch itself
// when the family's first kernel starts and its last kernel ends.
template <typename H>
void launch_hmom(const Fields<H> &f, const Consts &c, int wpb, int div, bool first, bool last, hipStream_t s,
                 hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
template <typename H>
void launch_vert(const Fields<H> &f, const Consts &c, int wpb, int div, bool first, bool stage_end, bool physics,
                 hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
template <typename H>
void launch_slow(const Fields<H> &f, const Consts &c, int wpb, bool from_t, hipStream_t s,
                 hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
template <typename H>
void launch_large(const Fields<H> &f, const Consts &c, int wpb, hipStream_t s, hipEvent_t ev0 = nullptr,
                  hipEvent_t ev1 = nullptr);
template <typename H>
void launch_diag_field(const Fields<H> &f, const Consts &c, int field, hipStream_t s);
// The checkpoint's fields into f.diag.
template <typename H>
void launch_export(const Fields<H> &f, const Consts &c, hipStream_t s);
// Per workgroup: largest speed and |w|, smallest and largest T of Phi[t].
template <typename H>
void launch_extremes(const Fields<H> &f, const Consts &c, double *out, hipStream_t s, int *nblocks_out);
template <typename H>
void launch_mass(const Fields<H> &f, const Consts &c, double *out, hipStream_t s, int *nblocks_out);
template <typename H>
void launch_to_state(const Fields<H> &f, const Consts &c, const double *blob, hipStream_t s);
// Total energy and mass partial sums of the state Phi[t] (which = 0) or of
// the small-step state (which = 1) into out[2 b], out[2 b + 1].
template <typename H>
void launch_energy(const Fields<H> &f, const Consts &c, int which, double *out, hipStream_t s, int *nblocks_out);
// Partial sums (one per workgroup) of the absolute axial angular momentum of
// the state Phi[t] (postproc.hip).
template <typename H>
void launch_angmom(const Fields<H> &f, const Consts &c, double *out, hipStream_t s, int *nblocks_out);
// The energy fixer after the dynamics of a large step (the start's partial
// sums already in f.epart), followed by the physics: replaces the physics of
// the last phase V, which then runs with last = false.
template <typename H>
void launch_fixer(const Fields<H> &f, const Consts &c, hipStream_t s);

// One member of an ensemble as the device sees it.
template <typename H>
struct Planet {
  Fields<H> f[2];   // the two buffer-set orders (see thor_state)
  Consts c;
};

enum class BatchOp { Large, Slow, Hmom, Vert, VertLast };

// Every member of an ensemble in one launch per phase.  arg0/arg1: Slow:
// from_t; Hmom: div, first | last << 1; Vert: div, first | stage_end << 1.
// max_cols: the most columns per wavefront of a member, of those that stage
// their stencil weights in LDS (at most kLdsCols).
template <typename H>
void launch_batch(const Planet<H> *P, const int2 *tiles, int n_tiles, int wpb, int parity, BatchOp op,
                  int arg0, int arg1, int max_cols, hipStream_t s);

}  // namespace thor
