// Internal declarations of the qeh library: context layout, FFT plans and the
// kernel launchers.  Not part of the public C ABI (include/qeh.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/qeh.h"

namespace qeh {

constexpr int kMaxPass = 8;
constexpr size_t kAlign = 256;
constexpr int kLdsMax = 160 * 1024;   // LDS per workgroup on gfx950

// Division by a fixed divisor d as q = (umulhi(n, m) + n) >> s, exact for
// n < 2^31 (round-up multiplier); built on the host, used in kernel index math.
struct FastDiv {
  uint32_t m, s, d;
};
FastDiv make_fastdiv(uint32_t d);

// One 1D mixed-radix transform of length n = prod radix[p].  Pass p combines
// radix[p] sub-transforms of length span[p] (span[0] = 1).  The decimation-
// in-time form takes digit-reversed input (element m at pos(m)) and returns
// natural order; the decimation-in-frequency form is its transpose.
struct FftDim {
  int n;
  int npass;
  int radix[kMaxPass];
  int span[kMaxPass];
  FastDiv nbf_div[kMaxPass];    // n / radix[p]
  FastDiv span_div[kMaxPass];   // span[p]
};

bool make_fft_dim(int n, FftDim *d);
// position of element m in the digit-reversed input of the DIT transform
int fft_digit_pos(const FftDim &d, int m);

// Plane-pass LDS geometry (elements of the working complex type).
struct PlaneGeom {
  int ldT;   // column stride of the x-extent column tile (>= N2, odd)
  int rc;    // rows processed together in the row phase
  int ldR;   // row stride of the row buffer (>= N1, odd)
  size_t lds_bytes;
  FastDiv ext_div, rc_div, rlast_div;   // ext, rc, rows of the last chunk
};

// Split plane path (planes too large for LDS): column groups of cg columns,
// row groups of rg rows (local column stride ldl).
struct SplitGeom {
  int cg, rg, ldl;
  size_t lds_col, lds_row;
  FastDiv cg_div, cglast_div, rg_div, rglast_div;
};

// Two-factor plane kernel (plane2.h): whether it runs, with unpadded columns or
// not, its column pitch, the split of a y position p into slot (p / b) * bp + p % b,
// rows at a time.
struct TwoGeom {
  int on, tight, half, rc, ldT, b, bp;
  size_t lds;
};

// Two-factor K1 / K3 (stick2.h): whether they run, 2^sl sticks per workgroup,
// line pitch, the split of a z position p into slot (p / b) * bp + p % b.
struct StickTwoGeom {
  int on, half, sl, ldz, b, bp;
  size_t lds;
};

struct StickGeom {
  int ldz;   // z-line stride (>= N3, odd)
  int S;     // sticks per workgroup
  size_t lds_bytes;
  FastDiv s_div, slast_div;   // S, sticks of the last workgroup
};

// Device arrays of one context, all inside the caller's arena.
struct DevMaps {
  int *stick_off;    // [nst+1] first G of each stick
  int *gmap;         // [npw] s*ldz + digit-reversed z position (two-factor K1 / K3:
                     // s * their pitch + slot)
  int *tidx;         // [nst] plane-tile index c*ldT + y-DIT input position of k mod N2
  int *tidx2;        // [nst] c*ldT + slot of k - kmin, for the two-factor plane kernel
  int *xin;          // [N1] column c whose h sits at x-DIT input position p, or -1
  double *kin;       // [npw] |k+G|^2
  double *hdiag;     // [npw] diag(H)
  void *vs;          // [N3][N2][N1] V/N (double or float)
  void *tw;          // twiddles x | y | z (double2 or float2)
  void *beta;        // [nkb][ldb] (double2 or float2)
  double2 *dmat;     // concatenated blocks
  double2 *qmat;     // overlap q blocks (same layout), or null
  int *pj0;          // [nkb] first projector of the atom block of i
  int *pnb;          // [nkb] size of that block
  int *pdoff;        // [nkb] offset of row i of its block in dmat
  int *chunk;        // [nchunk+1] atom-aligned projector ranges (<= 256 each)
  void *sbuf;        // [block][N3][nst] stick buffer (working complex type)
  void *part;        // [nsplit][block][nkb] split-K partials
  void *ps;          // [block][nkb] D * becp (working complex type; real floats on
                     // single-precision Gamma contexts)
  float2 *psi32;     // mixed form: [block][ldb] single-precision copy of psi (K1)
  void *big;         // split plane path: [block][N3][ext][N2] (or null)
  double2 *gbuf;     // Gamma, LDS-pass K3: [(block+1)/2][npw_fft] full-sphere H of band
                     // pairs (or null)
  int *colstart;     // [ext+1] first stick of each x-extent column
};

}  // namespace qeh

struct qeh_ctx {
  int npw = 0, nst = 0, nkb = 0, nat = 0;
  int npw_fft = 0;      // G-vectors of the FFT sphere (2 npw - 1 for Gamma cells, else npw)
  int gamma = 0;        // 1: real wavefunctions at k = 0, half sphere stored
  int has_q = 0;        // 1: overlap q blocks present (S != 1)
  int n1 = 0, n2 = 0, n3 = 0, ext = 0, hmin = 0;
  int block = 0, prec = 0;
  int plane_path = 0;   // 0 one kernel, 1 split through HBM; 2, 4: one kernel, names of box
                        // sizes only (qeh_ctx_info keeps them); which kernel: two.on
  int stick_path = 0;   // a name of sizes only as well; which kernel: st2.on
  int nsplit = 1, kchunk = 0;
  int form_proj = 0, form_expand = 0;   // FP64 beta^H psi and beta ps: GemmDesc::form, by block
  int wide = 0;         // 1: wide single-precision tiles for the projector products
  int ldb = 0;          // row length of beta and psi32 (npw; single precision: padded to
                        // whole 128-byte lines)
  int nchunk = 0;
  qeh::FftDim dx{}, dy{}, dz{};
  qeh::PlaneGeom pg{};
  qeh::SplitGeom spg{};
  qeh::StickGeom sg{};
  qeh::TwoGeom two{};
  qeh::StickTwoGeom st2{};
  int tw_off[3] = {0, 0, 0};
  hipStream_t stream = nullptr;
  qeh::DevMaps d{};
  char *arena = nullptr;
  size_t arena_bytes = 0;
  double vmean = 0.0;
  double omega = 0.0;   // cell volume
  // profiling
  bool prof = false;
  double stage_ms[QEH_NSTAGES] = {0};
  long stage_n[QEH_NSTAGES] = {0};
  std::vector<hipEvent_t> ev_pool;   // 2 events per recorded stage launch
  std::vector<int> ev_recs;          // stage id of each recorded launch
};

namespace qeh {

void set_error(const std::string &msg);
qeh_status hip_fail(hipError_t e, const char *what);

// ---- FFT path launchers (fft_kernels.hip) --------------------------------
// All take band count nbk (<= ctx block) and operate on the ctx stick buffer.
hipError_t launch_k1(const qeh_ctx *c, int nbk, const double2 *psi, int ldpsi);
// Gamma contexts: K1 of ceil(nbk/2) band pairs psi_2p + i psi_2p+1, read from
// the half-sphere bands (nbk rows, ldpsi) and expanded to the full sphere; with
// a device pair table, K1 of npairs pairs (rows pairs[p].x, pairs[p].y, the
// second < 0 for none).  copy32 (mixed form, natural pairs of a block of
// <= block bands): K1 also writes the block's single-precision copy psi32.
hipError_t launch_k1_gamma(const qeh_ctx *c, int nbk, const double2 *psi, int ldpsi,
                           const int2 *pairs = nullptr, int npairs = 0, bool copy32 = false);
hipError_t launch_k2(const qeh_ctx *c, int nbk);
// H psi of a block of nbk bands, local part, with the kinetic term.
hipError_t launch_k3(const qeh_ctx *c, int nbk, const double2 *psi, int ldpsi, double2 *hpsi,
                     int ldh);
// The two-factor forms (stick2_f32.hip, stick2_f64.hip): K1 of np bands or Gamma
// pairs (nbk, pairs: as in launch_k1_gamma); K3 as launch_k3.
hipError_t launch_k1_two_f32(const qeh_ctx *c, int np, const double2 *psi, int ldpsi, int nbk,
                             const int2 *pairs, float2 *psi32);
hipError_t launch_k1_two_f64(const qeh_ctx *c, int np, const double2 *psi, int ldpsi, int nbk,
                             const int2 *pairs, float2 *psi32);
hipError_t launch_k3_two_f32(const qeh_ctx *c, int nbk, const double2 *psi, int ldpsi,
                             double2 *hpsi, int ldh);
hipError_t launch_k3_two_f64(const qeh_ctx *c, int nbk, const double2 *psi, int ldpsi,
                             double2 *hpsi, int ldh);
// Their geometry for lines of n3 points holding l in [lmin, lmax]; false if n3
// is not a compiled size.
bool stick_two_geometry(int prec, int n3, int lmin, int lmax, StickTwoGeom *g);
size_t plane_lds_bytes(int prec, int ext, int n1, int n2, const PlaneGeom &g);
size_t stick_lds_bytes(int prec, int n3, const StickGeom &g);
// Square boxes that report plane path 2 or 4.
bool pair_plane_supported(int prec, int n1, int n2);
bool quad_plane_supported(int prec, int n1, int n2);

// Two-factor plane kernel: geometry for an x-extent of ext columns and a y
// extent of exty (false: no compiled form, or the columns leave too little LDS).
bool two_geometry(int prec, int n1, int n2, int ext, int exty, bool split, TwoGeom *g);
hipError_t launch_k2_two_f32(const qeh_ctx *c, int nbk);
hipError_t launch_k2_two_f64(const qeh_ctx *c, int nbk);

// Charge density: row groups of rg rows, subgroups of bsub bands.
struct DensityGeom {
  int rg, ngroups, bsub;
  bool pair;    // lane-pair rows kernel (partial planes in the same layout)
  bool fused;   // the two-factor plane kernel: no column pass through HBM
  size_t lds;
  FastDiv rg_div, rglast_div;
};
bool density_geometry(const qeh_ctx *c, DensityGeom *dg);
// One block of nbk bands whose sticks K1 has written: inverse y columns into
// big, then partial[sub][z][y][x] = sum over subgroup sub of occ_b |psi_b|^2.
hipError_t launch_density_columns(const qeh_ctx *c, int nbk, void *big);
// zcol: N2 zero complex values (single precision), read by the lane-pair rows
// for positions beyond the x-extent
hipError_t launch_density_rows(const qeh_ctx *c, const DensityGeom &dg, int nbk, const void *big,
                               const double *occ_d, double *partial, const void *zcol);
// Fused form (dg.fused): sticks -> columns -> rows -> partial planes in one pass.
hipError_t launch_density_plane(const qeh_ctx *c, const DensityGeom &dg, int nbk,
                                const double *occ_d, double *partial);
hipError_t launch_density_two_f32(const qeh_ctx *c, int nbk, int bsub, const double *occ,
                                  double *partial);
hipError_t launch_density_two_f64(const qeh_ctx *c, int nbk, int bsub, const double *occ,
                                  double *partial);
// LDS of the fused pass, 0 where it is not compiled.
size_t density_two_lds_f32(int n, int ext);
size_t density_two_lds_f64(int n, int ext);
hipError_t launch_density_reduce(const double *partial, int nsub, long npts, double scale,
                                 double *rho, int accumulate, hipStream_t s);

// ---- projectors built on the device (beta.cpp, beta_kernels.hip) -----------
// Workspace of the generator: the Miller list [npw][3] (in room for twice as
// much), per-atom int4 {species, first row, projectors, D offset}, positions
// [nat][3], channel offsets per species [nsp+1], l per channel, tables
// [channels][nq].
struct ProjgenLayout {
  size_t off_q, off_atom, off_tau, off_chan0, off_lchan, off_tab, total;
};
ProjgenLayout projgen_layout(const qeh_cell *c);   // c->projgen set
// Checks c->projgen against the cell (nproj per atom, table range over the
// sphere, finiteness); c's Miller list and lattice must already be valid.
qeh_status projgen_validate(const qeh_cell *c);
// Stages the generator inputs into work, writes beta (nkb rows of ldb complex,
// double2 if f64 else float2) and, when hdiag_dev is set, adds the nonlocal
// part of diag(H) (D blocks from dmat_dev); returns after the stream drained.
qeh_status projgen_run(const qeh_cell *c, bool f64, void *out, long ldb, char *work,
                       hipStream_t s, const double2 *dmat_dev, double *hdiag_dev);
// k and the reciprocal rows b[j] of the kernel's q = k + h b[0] + k b[1] + l b[2].
struct ProjgenFrame {
  double k[3], b[3][3];
};
hipError_t launch_beta_gen(bool f64, const int *miller, const ProjgenFrame &fr, int npw, int nat,
                           const int4 *atoms, const double *tau, const int *chan0,
                           const int *lchan, const double *tab, int nq, double dq, double pref,
                           void *beta, long ldb, hipStream_t s);
hipError_t launch_nl_diag(bool f64, const void *beta, long ldb, int npw, int nat,
                          const int4 *atoms, const double2 *dmat, double *hdiag,
                          hipStream_t s);
// Device address of the static staging array of qeh_beta_generate_static on
// the device of stream s (the current device when s is null); looked up once
// per device.
hipError_t beta_static_scratch(hipStream_t s, char **out);

// ---- complex GEMM launchers (gemm_kernels.hip) ----------------------------
// C[m][n] (+)= sum_k opA(A[m][k]) opB(B(k,n)), complex, MFMA.
//   A: element (m,k) at A[m*lda + k], conjugated if conjA.
//   B: bmode 0: element (k,n) at B[n*ldb + k] (conjugated if conjB);
//      bmode 1: element (k,n) at B[k*ldb + n].
//   Split-K: grid z = nsplit slices of kchunk; slice s writes
//      C + s*split_stride (accumulate must be 0 then).
enum GemmType { T_D2 = 0, T_F2 = 1, T_F1 = 2 };   // operand storage (T_F1: real float)
struct GemmDesc {
  const void *A; long lda; int ta;
  const void *B; long ldb; int tb; int bmode;
  void *C; long ldc; int tc;
  int M, N, K;
  int conjA, conjB, accumulate;
  int nsplit, kchunk; long split_stride;
  int tile;   // launch_split_gemm: 0 = 64 x 64, 1 = 64 x 128, 2 = 128 x 128
  int rmode;  // 0 complex; 1 only Re(C) wanted (Im written 0); 2 A real (Im A ignored)
  int form;   // launch_cgemm, complex: 3 or 4 real products (cgemm_form), 0 by this product's size
};
// FP64 operands and results.
hipError_t launch_cgemm(const GemmDesc &g, hipStream_t s);
// Whether launch_cgemm takes flat 16 x 64 tiles (else 64 x 64): callers that
// split K count their workgroups by it.
bool cgemm_flat(int M, int N, int K, int bmode);
// Real products of a complex one of this size: 4 (flat tiles) or 3.
int cgemm_form(int M, int N, int K, int bmode);
// The single-precision projector products: B and the products in single
// precision, beta^H psi (bmode 0, conjB; A in float or double, C float) and
// beta ps (bmode 1; C double).
hipError_t launch_split_gemm(const GemmDesc &g, hipStream_t s);

// ---- Davidson building blocks shared with the CG solver (davidson.cpp) ----
// out(i, j) = <X_i|Y_j> for i < nrow, j < ncol (col-major, ld), FP64 MFMA,
// split-K partials in `part` (room for part_cap of them) summed in a fixed order;
// real inner products on Gamma contexts.
hipError_t reduce_cols(const qeh_ctx *c, const double2 *X, int nrow, const double2 *Y, int ncol,
                       double2 *out, int ld, double2 *part, size_t part_cap);
// rows b < nb: out_b = sum_j Y(j, b) X_j  (Y col-major ld, j < n)
hipError_t rotate(const qeh_ctx *c, const double2 *Y, int ld, int n, int nb, const double2 *X,
                  double2 *out);
constexpr int kReduceMaxSplit = 32;

// ---- conjugate-gradient solver kernels (cg_kernels.hip) ----
// Slots of the solver's device scalar array (doubles; complex values take two).
enum CgSlot {
  kCgLam = 0,     // Rayleigh quotient of the current band
  kCgRR = 2,      // <r|r>
  kCgGpr = 4,     // <g_prev|r>
  kCgGam = 6,     // <g|r>
  kCgGamp = 8,    // previous <g|r>
  kCgXD = 10,     // <x|d>
  kCgDD = 12,     // <d|d>
  kCgB = 14,      // <x|H dn>
  kCgC = 16,      // <dn|H dn>
  kCgBeta = 18,   // conjugation factor
  kCgC0 = 20,     // rotation of (x, dn): c0 (real)
  kCgC1 = 22,     //   and c1 (complex)
  kCgInvD = 24,   // 1 / ||d - <x|d> x||
  kCgXX = 26,     // <x|x> at a band's start
  kCgInvX = 28,   // 1 / ||x||
  kCgFirst = 30,  // 1 on a band's first iteration
  kCgSlots = 32
};
constexpr int kCgDotBlocks = 64;   // stage-1 blocks per inner product
constexpr int kCgMaxDots = 4;      // inner products per launch
struct CgDots {
  const double2 *a[kCgMaxDots];
  const double2 *b[kCgMaxDots];
  int dst[kCgMaxDots];   // slot of <a|b> (re, im)
};
// inner products <a_q|b_q> into sc[dst_q] (part: 2 * kCgDotBlocks * npairs doubles)
hipError_t launch_cg_dots(const CgDots &p, int npairs, int npw, int gamma, double *part,
                          double *sc, hipStream_t s);
hipError_t launch_cg_resid(const double2 *x, const double2 *hx, const double *hdiag,
                           const double *sc, double2 *r, double2 *g, int npw, int gamma,
                           hipStream_t s);
hipError_t launch_cg_project(double2 *g, const double2 *X, long ldx, const double2 *coef, int m,
                             int npw, hipStream_t s);
hipError_t launch_cg_scale(double2 *x, const double *sc, int npw, hipStream_t s);
hipError_t launch_cg_dir(const double2 *g, double2 *d, double2 *gp, const double *sc, int npw,
                         hipStream_t s);
hipError_t launch_cg_dnorm(double2 *d, const double2 *x, double2 *dn, const double *sc, int npw,
                           hipStream_t s);
hipError_t launch_cg_update(double2 *x, double2 *hx, const double2 *dn, const double2 *hd,
                            const double *sc, int npw, hipStream_t s);
hipError_t launch_cg_scalar(double *sc, int phase, hipStream_t s);

// C[m][n] (+)= sum_s part[s*stride + m*ldp + n], summed in double in split order.
hipError_t launch_splitk_reduce(const void *part, int tp, long stride, int nsplit, int M, int N,
                                long ldp, double2 *C, long ldc, int accumulate, hipStream_t s);

// Sum split-K partials (double2 or float2 partials, double accumulation) and
// apply the block-diagonal D: ps[b][i] = sum_j D_ij sum_s part[s][b][j].
// Gamma contexts: psi (ldpsi) are the block's bands, whose G = 0 values enter
// the real full-sphere projection (ignored otherwise).
// mat: the block-diagonal matrix applied (D, or the overlap's q; null = D).
hipError_t launch_dscale(const qeh_ctx *c, int nbk, const double2 *psi, long ldpsi,
                         const double2 *mat = nullptr);

// ---- dense Hermitian subspace solver (eigh_kernels.hip) --------------------
// Reduced problems up to kEigMaxN; column-major double2 matrices.
constexpr int kEigMaxN = 2048;
// Orders that the one-workgroup kernels of eigh_small.hip hold in registers.
constexpr int kEigRegN = 128;
// Largest basis for which the Davidson's automatic choice takes the own solver:
// above it the one-stage Householder reduction streams the trailing matrix
// from HBM at every step (n = 2048: 86 ms per complex solve) and rocSOLVER's
// real solver of the Gamma path measured faster (512-atom cell: 12.8 against
// 13.6 s per Davidson run).
constexpr int kEigAutoMaxN = 1024;
// The solver's launchers take `wide`: true spreads each step over many
// workgroups (shortest time for one solve alone on the device), false keeps
// the Cholesky, the Householder reduction and the bisection on one workgroup
// each (least device time, for solves that share the device with others).
// S = L L^H in place (lower); info = 0 or the failing column + 1.  scr: 64 n
// doubles of scratch (the eigenpair scratch below is large enough and free).
hipError_t launch_chol(double2 *S, long ld, int n, int *info, double *scr, bool wide,
                       hipStream_t s);
// The same and the tridiagonalisation for orders <= kEigRegN (eigh_small.hip).
hipError_t launch_chol_reg(double2 *S, long ld, int n, int *info, hipStream_t s);
hipError_t launch_tridiag_reg(double2 *A, long lda, int m, double *d, double *e, double2 *tau,
                              const int *info_chol, hipStream_t s);
// launch_trsm and launch_backtr (below) for orders <= 256.
hipError_t launch_trsm_small(int mode, const double2 *T, long ldt, int n, const double2 *B,
                             long ldb, int ncol, double2 *X, long ldx, hipStream_t s);
hipError_t launch_backtr_small(const double2 *A, long lda, int n, const double *tri,
                               const double *Zt, int ldz, int nb, double2 *Zc, long ldc,
                               const int *info_chol, const int *info_eig, hipStream_t s);
// X = L^-1 B (mode 0, T = L lower), X = L^-1 M^H with B = M (mode 1), or
// X = U^-1 B (mode 2, T = U upper, backward); ncol columns, one wave each.
hipError_t launch_trsm(int mode, const double2 *T, long ldt, int n, const double2 *B, long ldb,
                       int ncol, double2 *X, long ldx, hipStream_t s);
// A = Q T Q^H (Householder, in place); tri = d[n] | e[n] | tau (double2)[n].
// scr: 12 n doubles of scratch (the multi-workgroup steps' vectors); the
// eigenpair scratch below is large enough and free at this point.
hipError_t launch_tridiag(double2 *A, long lda, int n, double *tri, double *scr,
                          const int *info_chol, bool wide, hipStream_t s);
// nb lowest eigenpairs of T: w[nb] ascending, Z (real, n x nb, ldz); scr holds
// eig_scratch_doubles(n) doubles; info 0 / nonzero on failure.
size_t eig_scratch_doubles(int n);
hipError_t launch_trieig(const double *tri, int n, int nb, double *w, double *Z, int ldz,
                         double *scr, int *info, const int *info_chol, bool wide, hipStream_t s);
// Zc = Q Zt (n x nb) through the reflectors stored in A by launch_tridiag.
hipError_t launch_backtr(const double2 *A, long lda, int n, const double *tri, const double *Zt,
                         int ldz, int nb, double2 *Zc, long ldc, const int *info_chol,
                         const int *info_eig, hipStream_t s);

// ---- Davidson helpers (dav_kernels.hip) ----------------------------------
// norms[b] = || Q_b - eps_b P_b ||^2 over npw (double), one launch; gamma = 1:
// half-sphere vectors, every G != 0 counted twice (G and -G).
hipError_t launch_resid_norms(const double2 *P, const double2 *Q, long ld, int npw,
                              int nb, const double *eps, double *norms, int gamma,
                              hipStream_t s);
// V[dst_b] = t / ||t||, t = (Q_b - eps_b P_b) / sqrt(1 + (h - eps_b)^2) for the
// listed bands b = idx[j], dst row j (norm as above).
hipError_t launch_precond(const double2 *P, const double2 *Q, long ld, int npw,
                          const int *idx, int nc, const double *eps, const double *hdiag,
                          double2 *V, long ldv, int gamma, hipStream_t s);
// Gamma point (real wavefunctions, half sphere of nh coefficients, G = 0 first):
// split the full-sphere result (2 nh - 1 entries, -G before G) of the local
// operator on band pairs psi_2p + i psi_2p+1 back into the two bands (+ kinetic
// term), writing hpsi.
hipError_t launch_gamma_unpack(const double2 *hc, long ldc, int nbk, int nh, const double2 *psi,
                               long ldpsi, const double *kin, double2 *hpsi, long ldh,
                               hipStream_t s);
// M(i, j) <- 2 Re M(i, j) - Re X_i[0] Re Y_j[0] (imaginary part zero): half-sphere
// sums turned into full-sphere inner products of real functions.
hipError_t launch_gamma_inner(double2 *M, long ld, int nrow, int ncol, const double2 *X,
                              const double2 *Y, long npw, hipStream_t s);
hipError_t launch_zero_g0_imag(double2 *psi, long ldpsi, int nb, hipStream_t s);
// n x n blocks, column-major: R = Re M, and M = R + 0 i.
hipError_t launch_real_part(const double2 *M, long ld, double *R, long ldr, int n,
                            hipStream_t s);
hipError_t launch_real_to_complex(const double *R, long ldr, double2 *M, long ld, int n,
                                  hipStream_t s);
// Copy rows; Hermitian fill; diag set etc.
hipError_t launch_copy_rows(const double2 *src, long lds, double2 *dst, long ldd, int npw,
                            int nrows, hipStream_t s);
// M[j][i] = conj(M[i][j]) for i in [0,n0), j in [n0,n1) (col-major, ld): fills
// the rows n0..n1 of the first n0 columns from the new columns.
hipError_t launch_herm_fill(double2 *M, long ld, int n0, int n1, hipStream_t s);
// M[0:n,0:n] = diag(d) (complex), or identity if d == null.
hipError_t launch_set_diag(double2 *M, long ld, int n, const double *d, hipStream_t s);
// dst (n x n, ldd) = (src + src^H)/2 (src n x n, lds), col-major.
hipError_t launch_hermitise_copy(const double2 *src, long lds, double2 *dst, long ldd, int n,
                                 hipStream_t s);
// L = lower triangle of M (zeros above), LH = L^H; all n x n col-major, ld.
hipError_t launch_tril_adjoint(const double2 *M, double2 *L, double2 *LH, long ld, int n,
                               hipStream_t s);
// p[0..n) = v (a kernel, not a memset, so the call can sit in captured graphs)
hipError_t launch_fill_int(int *p, int n, int v, hipStream_t s);
// finite check: flag[0] |= any non-finite in x[0..n) (doubles)
hipError_t launch_check_finite(const double *x, long n, int *flag, hipStream_t s);

}  // namespace qeh
