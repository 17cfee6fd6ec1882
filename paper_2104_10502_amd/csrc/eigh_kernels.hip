// Dense Hermitian solver of the Davidson Rayleigh-Ritz step, written for the
// small reduced problems of block Davidson (n <= 2048): the paper solves this
// small generalized eigenproblem with a dense GPU solver (section "Evolution
// of the GPU-enabled version").  H y = eps S y for the lowest nb
// pairs, in deterministic kernels (fixed summation orders, no atomics on
// floating-point data):
//
//   chol_reg_kernel (eigh_small.hip) one workgroup, orders <= 128: S = L L^H,
//                   the matrix in registers; above it chol_kernel (one
//                   workgroup) or cholp_kernel (one launch per 16-column panel
//                   over many workgroups)
//   trsm_kernel     one wave per column, many workgroups: L X = B (forward),
//                   with B given or as the adjoint of a matrix, or L^H X = B
//                   (backward with the explicit L^H); A = L^-1 H L^-H by two
//                   of them, Y = L^-H Z by a third
//   tdstep_kernel   one launch per Householder step while the trailing block
//                   is larger than kTailN, one wave per column, many
//                   workgroups
//   tridiag_reg_kernel  (eigh_small.hip) one workgroup, trailing block in
//                   registers: the last kTailN steps of the Householder reduction A = Q T Q^H, T
//                   real symmetric tridiagonal (d, e), reflectors kept in A
//   trieig_kernel   the nb lowest eigenpairs of T.  T is split where
//                   |e_k| <= eps ||T||; the global nb-th eigenvalue is
//                   bracketed by multisection of Sturm counts; every block's
//                   eigenvalues below it are found by multisection over many
//                   workgroups (first launch) and sorted (second launch, one
//                   workgroup); eigenvectors come from twisted
//                   factorizations of T_b - lambda I (one thread each), except
//                   for groups of numerically equal eigenvalues of one block
//                   (gap <= 1e-12 ||T||, as exact multiplets of A leave them:
//                   Householder does not split T there), which get inverse
//                   iteration from distinct start vectors through one pivoted
//                   LU of T_b - sigma I with Gram-Schmidt between the two
//                   sweeps; vectors of close eigenvalues of one block
//                   (gap <= 1e-5 ||T||) are re-orthogonalised in index order
//   backtr_kernel   one wave per column, many workgroups: Z = Q Z_T through
//                   the stored reflectors (staged in LDS, shared by a
//                   workgroup's waves)
//
// Storage: column-major double2 matrices with leading dimension ld.  A real
// symmetric pair (Gamma point) goes through the same kernels with zero
// imaginary parts, which stay zero.
#include "eigh_vec.h"

namespace qeh {
namespace {

constexpr int kCholMaxN = 512;       // largest order of the one-workgroup Cholesky (LDS panel)

// ---------------------------------------------------------------- Cholesky
// S (n x n, lower triangle read) = L L^H in place (lower).  info = 0, or
// j + 1 if the leading (j+1) x (j+1) minor is not positive definite (or not
// finite); L is then incomplete.
//
// Right-looking by panels of kCB columns: the panel (rows jb..n-1) is
// factored in LDS, written back, and the trailing lower triangle gets one
// rank-kCB update, each element read and written once per panel (the row's
// panel entries in registers, the column's broadcast from LDS).
constexpr int kCB = 16;
constexpr int kCBP = kCB + 1;   // padded LDS row stride (bank spread)

__global__ __launch_bounds__(kET) void chol_kernel(double2 *S, long ld, int n, int *info) {
  __shared__ double2 P[kCholMaxN * kCBP];
  const int tid = threadIdx.x;
  for (int jb = 0; jb < n; jb += kCB) {
    const int b = min(kCB, n - jb), m = n - jb;
    for (int idx = tid; idx < m * kCB; idx += kET) {
      const int r = idx % m, c = idx / m;
      P[r * kCBP + c] = (c < b && r >= c) ? S[(jb + r) + (long)(jb + c) * ld] : make_double2(0.0, 0.0);
    }
    __syncthreads();
    for (int c = 0; c < b; ++c) {
      const double ajj = P[c * kCBP + c].x;
      if (!(ajj > 0.0) || !isfinite(ajj)) {   // same value in every thread
        if (tid == 0) *info = jb + c + 1;
        return;
      }
      const double ljj = sqrt(ajj), rinv = 1.0 / ljj;
      __syncthreads();
      for (int r = c + tid; r < m; r += kET)
        P[r * kCBP + c] = r == c ? make_double2(ljj, 0.0) : cscale(P[r * kCBP + c], rinv);
      __syncthreads();
      const int w = b - c - 1;
      for (int idx = tid; idx < m * w; idx += kET) {
        const int r = idx % m, c2 = c + 1 + idx / m;
        if (r >= c2) P[r * kCBP + c2] = csub(P[r * kCBP + c2], cmulc(P[r * kCBP + c], P[c2 * kCBP + c]));
      }
      __syncthreads();
    }
    for (int idx = tid; idx < m * b; idx += kET) {
      const int r = idx % m, c = idx / m;
      if (r >= c) S[(jb + r) + (long)(jb + c) * ld] = P[r * kCBP + c];
    }
    const int mt = n - jb - b;
    if (mt > 0) {
      const int g = kET / mt;   // >= 2
      if (tid < g * mt) {
        const int r = tid % mt, grp = tid / mt;
        double2 pr[kCB];
#pragma unroll
        for (int c = 0; c < kCB; ++c) pr[c] = P[(b + r) * kCBP + c];
        double2 *row = S + (jb + b + r) + (long)(jb + b) * ld;
        for (int kk = grp; kk <= r; kk += g) {
          const double2 *pk = P + (b + kk) * kCBP;
          double2 acc = row[(long)kk * ld];
#pragma unroll
          for (int c = 0; c < kCB; ++c) acc = csub(acc, cmulc(pr[c], pk[c]));
          row[(long)kk * ld] = acc;
        }
      }
    }
    __syncthreads();
  }
  if (tid == 0) *info = 0;
}

// Blocked form over many workgroups, one launch per panel of kCB columns.
// Launch p (panel jb = p kCB): every workgroup factors the b x b diagonal
// block L11 itself (the same data and arithmetic in each, hence the same
// L11), forms the rows of L21 = A21 L11^-H that its kCT x kCT tile of the
// trailing lower triangle needs, and subtracts L21 L21^H from that tile.  The
// factored panel goes to a scratch panel (parity p & 1; L11 by tile (0, 0),
// the rows of L21 by the diagonal tiles) and launch p + 1, which reads
// neither, copies it into S: within a launch no workgroup writes what another
// reads.  The last panel (no trailing block) writes its L11 to S itself.
// Launch 0 sets info = 0; a panel that is not positive definite sets
// jb + c + 1, and every later launch returns at once.
constexpr int kCT = 32;   // trailing-update tile

__global__ __launch_bounds__(256) void cholp_kernel(double2 *S, long ld, int n, int jb,
                                                    double2 *scr, int *info) {
  __shared__ double2 D[kCB * kCBP];          // diagonal block -> L11
  __shared__ double2 Lr[2][kCT * kCBP];      // panel rows of the tile's rows / columns
  const int tid = threadIdx.x;
  if (jb > 0 && *info != 0) return;
  if (jb == 0 && blockIdx.x == 0 && tid == 0) *info = 0;
  const int b = min(kCB, n - jb), m = n - jb, mt = m - b;
  const int pan = jb / kCB;
  double2 *cur = scr + (long)(pan & 1) * n * kCB;
  // the previous panel into S
  if (jb > 0) {
    const int jp = jb - kCB, mp = n - jp;
    const double2 *prev = scr + (long)((pan - 1) & 1) * n * kCB;
    for (int idx = blockIdx.x * 256 + tid; idx < mp * kCB; idx += gridDim.x * 256) {
      const int r = idx % mp, c = idx / mp;
      if (r >= c) S[(jp + r) + (long)(jp + c) * ld] = prev[r * kCB + c];
    }
  }
  for (int idx = tid; idx < kCB * kCB; idx += 256) {
    const int r = idx % kCB, c = idx / kCB;
    D[r * kCBP + c] = (r < b && c < b && r >= c) ? S[(jb + r) + (long)(jb + c) * ld]
                                                : make_double2(0.0, 0.0);
  }
  __syncthreads();
  for (int c = 0; c < b; ++c) {
    const double ajj = D[c * kCBP + c].x;
    if (!(ajj > 0.0) || !isfinite(ajj)) {   // same value in every workgroup
      if (blockIdx.x == 0 && tid == 0) *info = jb + c + 1;
      return;
    }
    const double ljj = sqrt(ajj), rinv = 1.0 / ljj;
    __syncthreads();
    if (tid >= c && tid < b)
      D[tid * kCBP + c] = tid == c ? make_double2(ljj, 0.0) : cscale(D[tid * kCBP + c], rinv);
    __syncthreads();
    const int w = b - c - 1;
    if (tid < b * w) {
      const int r = tid % b, c2 = c + 1 + tid / b;
      if (r >= c2) D[r * kCBP + c2] = csub(D[r * kCBP + c2], cmulc(D[r * kCBP + c], D[c2 * kCBP + c]));
    }
    __syncthreads();
  }
  if (mt == 0) {   // last panel
    if (blockIdx.x == 0)
      for (int idx = tid; idx < b * b; idx += 256) {
        const int r = idx % b, c = idx / b;
        if (r >= c) S[(jb + r) + (long)(jb + c) * ld] = D[r * kCBP + c];
      }
    return;
  }
  // this workgroup's tile (ti >= tj) of the trailing lower triangle
  const int x = blockIdx.x;
  int ti = (int)((sqrt(8.0 * x + 1.0) - 1.0) * 0.5);
  while (ti * (ti + 1) / 2 > x) --ti;
  while ((ti + 1) * (ti + 2) / 2 <= x) ++ti;
  const int tj = x - ti * (ti + 1) / 2;
  const int r0[2] = {ti * kCT, tj * kCT};   // rows of the trailing block
  // panel rows of the tile's rows and columns, then L21 = A21 L11^-H (one
  // thread per row, forward in the column index)
  for (int idx = tid; idx < 2 * kCT * kCB; idx += 256) {
    const int h = idx / (kCT * kCB), e = idx % (kCT * kCB);
    const int r = e % kCT, c = e / kCT;
    const int gr = r0[h] + r;
    Lr[h][r * kCBP + c] = (gr < mt && c < b) ? S[(jb + b + gr) + (long)(jb + c) * ld]
                                             : make_double2(0.0, 0.0);
  }
  __syncthreads();
  if (tid < 2 * kCT) {
    const int h = tid / kCT, r = tid % kCT;
    double2 *row = &Lr[h][r * kCBP];
    for (int c = 0; c < b; ++c) {
      double2 a = row[c];
      for (int c2 = 0; c2 < c; ++c2) a = csub(a, cmulc(row[c2], D[c * kCBP + c2]));
      row[c] = cscale(a, 1.0 / D[c * kCBP + c].x);
    }
  }
  __syncthreads();
  // the factored panel to the scratch panel
  if (ti == tj) {
    for (int idx = tid; idx < kCT * kCB; idx += 256) {
      const int r = idx % kCT, c = idx / kCT;
      if (r0[0] + r < mt) cur[(b + r0[0] + r) * kCB + c] = Lr[0][r * kCBP + c];
    }
    if (ti == 0)
      for (int idx = tid; idx < kCB * kCB; idx += 256) {
        const int r = idx % kCB, c = idx / kCB;
        cur[r * kCB + c] = D[r * kCBP + c];
      }
  }
  // tile -= L21(rows) L21(cols)^H
  for (int e = tid; e < kCT * kCT; e += 256) {
    const int r = e % kCT, k = e / kCT;
    const int gr = r0[0] + r, gk = r0[1] + k;
    if (gr >= mt || gk >= mt || gk > gr) continue;
    double2 *p = S + (jb + b + gr) + (long)(jb + b + gk) * ld;
    double2 acc = *p;
#pragma unroll
    for (int c = 0; c < kCB; ++c) acc = csub(acc, cmulc(Lr[0][r * kCBP + c], Lr[1][k * kCBP + c]));
    *p = acc;
  }
}

// ---------------------------------------------------------------- tridiagonalisation
// A (n x n Hermitian, full storage) = Q T Q^H, Q = H_0 ... H_{n-2},
// H_k = I - tau_k v_k v_k^H acting on rows k+1..n-1.  On return column k of A
// holds v_k in rows k+1..n-1 (v_k[k+1] = 1); tri = d[n] | e[n] | tau (double2)[n].
//
// Step k needs p = A22 v_k (A22 = rows / columns k+1..) and applies the
// rank-2 update A22 -= v w^H + w v^H.
//
// Householder vector of the column col[0..m) (col[0] the subdiagonal entry):
// tau, beta, and v written to col (v[0] = 1) and to vs.  Uniform in all NT
// threads of the workgroup.
template <int NT = kET>
__device__ void householder(double2 *col, int m, double2 *vs, double *red, double2 *t_out,
                            double *beta_out) {
  const int tid = threadIdx.x;
  // alpha is read before the barriers of the sum: thread 0 overwrites col[0]
  // with v[0] = 1 below, and a wave that read it only after the sum could
  // see that write
  double2 alpha = col[0];
  auto norm2 = [&](double up) {   // of the entries below, scaled by up
    double s = 0.0;
    for (int i = 1 + tid; i < m; i += NT) {
      const double2 v = cscale(col[i], up);
      s += v.x * v.x + v.y * v.y;
    }
    return block_sum<NT / 64>(s, red);
  };
  double up = 1.0, xn2 = norm2(up);
  if (alpha.x * alpha.x + alpha.y * alpha.y + xn2 < 0x1p-900) {
    up = 0x1p500;   // uniform; the squares would lose their digits
    alpha = cscale(alpha, up);
    xn2 = norm2(up);
  }
  double beta;
  double2 t = make_double2(0.0, 0.0), scale = make_double2(0.0, 0.0);
  if (xn2 == 0.0 && alpha.y == 0.0) {
    beta = alpha.x;
  } else {
    beta = -copysign(sqrt(alpha.x * alpha.x + alpha.y * alpha.y + xn2), alpha.x);
    t = make_double2((beta - alpha.x) / beta, -alpha.y / beta);
    const double2 ab = make_double2(alpha.x - beta, alpha.y);
    const double den = ab.x * ab.x + ab.y * ab.y;
    scale = make_double2(up * (ab.x / den), -up * (ab.y / den));   // 1 / (alpha - beta)
  }
  beta /= up;
  const bool refl = t.x != 0.0 || t.y != 0.0;
  for (int i = tid; i < m; i += NT) {
    const double2 v = i == 0 ? make_double2(1.0, 0.0) : (refl ? cmul(col[i], scale) : col[i]);
    vs[i] = v;
    col[i] = v;
  }
  *t_out = t;
  *beta_out = beta;
}

constexpr int kTU = 6;   // independent loads in flight per thread

// One pass over the m x m block U (columns 1..m-1, rows 1..m-1 of the
// trailing matrix of step k; element (i, j) at U[i + j*lda]):
//   if upd:  U(i, j) -= v_i conj(w_j) + w_i conj(v_j)   (stored back)
//   if vn:   part[grp * mm + (i - 1)] = sum over the thread's columns of U(i, j) vn_{j-1}
// Rows and columns 0 (column 0 was done separately) are skipped.
__device__ void fused_pass(double2 *U, long lda, int m, bool upd, const double2 *vs,
                           const double2 *ws, bool mv, const double2 *vn, double2 *part) {
  const int tid = threadIdx.x;
  const int mm = m - 1;
  if (mm <= 0) return;
  const int g = kET / mm;   // >= 1 (mm < kEMaxN)
  if (tid >= g * mm) return;
  const int r = tid % mm, grp = tid / mm;
  const int i = r + 1;
  const double2 vi = vs[i], wi = ws[i];
  double2 acc = make_double2(0.0, 0.0);
  int j = 1 + grp;
  for (; j + (kTU - 1) * g < m; j += kTU * g) {
    double2 a[kTU];
#pragma unroll
    for (int u = 0; u < kTU; ++u) a[u] = U[i + (long)(j + u * g) * lda];
#pragma unroll
    for (int u = 0; u < kTU; ++u) {
      const int jj = j + u * g;
      if (upd) {
        a[u] = csub(a[u], cadd(cmulc(vi, ws[jj]), cmulc(wi, vs[jj])));
        U[i + (long)jj * lda] = a[u];
      }
      if (mv) acc = cadd(acc, cmul(a[u], vn[jj - 1]));
    }
  }
  for (; j < m; j += g) {
    double2 a = U[i + (long)j * lda];
    if (upd) {
      a = csub(a, cadd(cmulc(vi, ws[j]), cmulc(wi, vs[j])));
      U[i + (long)j * lda] = a;
    }
    if (mv) acc = cadd(acc, cmul(a, vn[j - 1]));
  }
  if (mv) part[grp * mm + r] = acc;
}

// The whole reduction on one workgroup, the trailing matrix streamed from
// memory once per step (rank-2 update of step k fused with the product of
// step k+1): little device time in total, for solves that share the device.
__global__ __launch_bounds__(kET) void tridiag_kernel(double2 *A, long lda, int n, double *d,
                                                      double *e, double2 *tau,
                                                      const int *info_chol) {
  if (*info_chol != 0) return;
  __shared__ double2 vbuf[2][kEMaxN];   // v_k and v_{k+1}
  __shared__ double2 ps[kEMaxN];        // A22 v_k, then p, then w
  __shared__ double2 part[kET];
  __shared__ double red[kEW];
  const int tid = threadIdx.x;
  if (n == 1) {
    if (tid == 0) d[0] = A[0].x;
    return;
  }
  // step 0's reflector and its product A22 v_0 (a plain pass: no update)
  double2 t;
  double beta;
  householder(A + 1, n - 1, vbuf[0], red, &t, &beta);
  if (tid == 0) {
    d[0] = A[0].x;
    e[0] = beta;
    tau[0] = t;
  }
  __syncthreads();
  {
    // the pass skips row / column 0 of its block: hand it the whole A22 by
    // starting one row and column earlier (A11 corner of A)
    const int m = n - 1;
    // rows 0..m-1 of A22 times v: do row 0 and column 0 here too
    const double2 *a22 = A + lda + 1;
    const int g = kET / m;
    if (tid < g * m) {
      const int i = tid % m, grp = tid / m;
      double2 acc = make_double2(0.0, 0.0);
      int jj = grp;
      for (; jj + (kTU - 1) * g < m; jj += kTU * g) {
        double2 a[kTU];
#pragma unroll
        for (int u = 0; u < kTU; ++u) a[u] = a22[i + (long)(jj + u * g) * lda];
#pragma unroll
        for (int u = 0; u < kTU; ++u) acc = cadd(acc, cmul(a[u], vbuf[0][jj + u * g]));
      }
      for (; jj < m; jj += g) acc = cadd(acc, cmul(a22[i + (long)jj * lda], vbuf[0][jj]));
      part[tid] = acc;
    }
    __syncthreads();
    for (int i = tid; i < m; i += kET) {
      double2 acc = part[i];
      for (int q = 1; q < g; ++q) acc = cadd(acc, part[q * m + i]);
      ps[i] = acc;
    }
    __syncthreads();
  }
  int cur = 0;
  for (int k = 0; k + 1 < n; ++k) {
    const int m = n - k - 1;   // order of A22 of step k
    double2 *u = A + (long)(k + 1) * lda + (k + 1);   // A22 of step k, (0, 0) corner
    const double2 *vs = vbuf[cur];
    const bool refl = t.x != 0.0 || t.y != 0.0;
    if (refl) {
      // p = t A22 v, alpha2 = -1/2 t (p^H v), w = p + alpha2 v (in ps)
      double dr = 0.0, di = 0.0;
      for (int i = tid; i < m; i += kET) {
        const double2 p = cmul(t, ps[i]), v = vs[i];
        dr += p.x * v.x + p.y * v.y;
        di += p.x * v.y - p.y * v.x;
      }
      dr = block_sum(dr, red);
      di = block_sum(di, red);
      const double2 a2 = cscale(cmul(t, make_double2(dr, di)), -0.5);
      for (int i = tid; i < m; i += kET) ps[i] = cadd(cmul(t, ps[i]), cmul(a2, vs[i]));
      __syncthreads();
      // column 0 of A22 (column k+1 of A), rows 0..m-1
      for (int i = tid; i < m; i += kET)
        u[i] = csub(u[i], cadd(cmulc(vs[i], ps[0]), cmulc(ps[i], vs[0])));
      __syncthreads();
    }
    if (m == 1) {
      if (tid == 0) d[k + 1] = u[0].x;
      break;
    }
    // reflector of step k+1 from column k+1 below the diagonal
    double2 t1;
    double beta1;
    householder(u + 1, m - 1, vbuf[cur ^ 1], red, &t1, &beta1);
    if (tid == 0) {
      d[k + 1] = u[0].x;
      e[k + 1] = beta1;
      tau[k + 1] = t1;
    }
    __syncthreads();
    const bool refl1 = t1.x != 0.0 || t1.y != 0.0;
    // rest of step k's update fused with step k+1's product (rows / columns
    // 1..m-1 of this A22 are A22 of step k+1)
    fused_pass(u, lda, m, refl, vs, ps, refl1, vbuf[cur ^ 1], part);
    __syncthreads();
    if (refl1) {
      const int mm = m - 1, g = kET / mm;
      for (int i = tid; i < mm; i += kET) {
        double2 acc = part[i];
        for (int q = 1; q < g; ++q) acc = cadd(acc, part[q * mm + i]);
        ps[i] = acc;
      }
    }
    __syncthreads();
    t = t1;
    cur ^= 1;
  }
}

// Leading steps of the same reduction while the trailing block is large: one
// launch per step over many workgroups, one wave per column of the trailing
// block (kSW columns per workgroup); tridiag_reg_kernel then reduces the last
// kTailN rows and columns as a problem of its own (after k0 steps the rest of
// the reduction is the reduction of the updated block A[k0:, k0:]).
//
// Launch k (k = -1 .. k0-1) applies step k's update A22 -= v w^H + w v^H
// (A22 = rows / columns k+1..n-1) to the columns its waves own, and forms
// step k+1's reflector v' (from column k+1) and product y' = A22' v' (A22' =
// rows / columns k+2..) for the next launch.  w needs the whole y of step k,
// and v' the updated column k+1: every workgroup forms both itself from the
// small vectors of the previous launch (the same arithmetic in each, hence
// the same values), so the launch boundary is the only synchronisation.  y'
// uses the Hermitian symmetry, (A22' v')_j = sum_i conj(A(i, j)) v'_i, so
// that a wave needs only its own column.  Launch -1 only forms v_0 and y_0.
// Scratch (double2, double-buffered by parity so that a launch never writes
// what it reads): vb[2][n] = v of a step, yb[2][n] = its y, cb[2][n] =
// column c of A (rows c..n-1) as the launch before left it, for c = k+1.
// Column k's reflector is written into A by the launch of step k, when no
// wave reads that column any more.
constexpr int kSW = 4;         // waves (columns) per workgroup of the step kernel
constexpr int kTailN = kEigRegN;   // order left to the one-workgroup kernel

template <int NS>   // register slots per lane: orders up to 64 NS
__global__ __launch_bounds__(64 * kSW) void tdstep_kernel(double2 *A, long lda, int n, int k,
                                                          int last, double *d, double *e,
                                                          double2 *tau, double2 *scr,
                                                          const int *info_chol) {
  if (*info_chol != 0) return;
  __shared__ double2 vs[NS * 64];   // v of step k
  __shared__ double2 ws[NS * 64];   // y of step k, then w
  __shared__ double2 cs[NS * 64];   // column k+1 (rows k+1..), then v' in cs[1..]
  __shared__ double red[2 * kSW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int r0 = k + 1;            // first row / column of A22
  const int m = n - r0;            // its order
  double2 *vb = scr, *yb = scr + 2 * (long)n, *cb = scr + 4 * (long)n;
  const int col = blockIdx.x * kSW + (tid >> 6);   // this wave's column of A22
  const bool own = col < m;
  double2 *acol = A + (long)(r0 + col) * lda + r0;
  // the owned column first: its loads overlap the small vectors'
  double2 a[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = s * 64 + lane;
    a[s] = own && i < m ? acol[i] : make_double2(0.0, 0.0);
  }
  const double2 t = k >= 0 ? tau[k] : make_double2(0.0, 0.0);
  const bool refl = t.x != 0.0 || t.y != 0.0;
  const double2 *csrc = k >= 0 ? cb + (long)(r0 & 1) * n : A;
  for (int i = tid; i < m; i += 64 * kSW) {
    if (k >= 0) {
      vs[i] = vb[(long)(k & 1) * n + i];
      ws[i] = yb[(long)(k & 1) * n + i];
    }
    cs[i] = csrc[i];
  }
  __syncthreads();
  if (refl) {
    // p = t y, alpha = -1/2 t (p^H v), w = p + alpha v; then column k+1
    // less v w0^* + w v0^*.  Every thread forms w0 itself from y0 and v0,
    // read before the sum's barriers (thread 0 overwrites ws[0] with w0 below).
    const double2 y0 = ws[0], v0 = vs[0];
    double dr = 0.0, di = 0.0;
    for (int i = tid; i < m; i += 64 * kSW) {
      const double2 p = cmul(t, ws[i]), v = vs[i];
      dr += p.x * v.x + p.y * v.y;
      di += p.x * v.y - p.y * v.x;
    }
    const double2 pv = block_sum2<kSW>(dr, di, red);
    const double2 a2 = cscale(cmul(t, pv), -0.5);
    const double2 w0 = cadd(cmul(t, y0), cmul(a2, v0));
    for (int i = tid; i < m; i += 64 * kSW) {
      const double2 wi = cadd(cmul(t, ws[i]), cmul(a2, vs[i]));
      ws[i] = wi;
      cs[i] = csub(cs[i], cadd(cmulc(vs[i], w0), cmulc(wi, v0)));
    }
    __syncthreads();
  }
  double2 t1 = make_double2(0.0, 0.0);
  double beta1 = 0.0;
  if (!last) {
    householder<64 * kSW>(cs + 1, m - 1, cs + 1, red, &t1, &beta1);
    __syncthreads();
  }
  if (own) {
    if (refl) {
      const double2 vj = vs[col], wj = ws[col];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int i = s * 64 + lane;
        if (i < m) {
          a[s] = csub(a[s], cadd(cmulc(vs[i], wj), cmulc(ws[i], vj)));
          acol[i] = a[s];
        }
      }
    }
    if (!last && col >= 1) {
      double dr = 0.0, di = 0.0;   // conj(column) . v'
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int i = s * 64 + lane;
        if (i >= 1 && i < m) {
          const double2 v = cs[i];
          dr += a[s].x * v.x + a[s].y * v.y;
          di += a[s].x * v.y - a[s].y * v.x;
        }
      }
      dr = wave_sum(dr);
      di = wave_sum(di);
      if (lane == 0) yb[(long)(r0 & 1) * n + col - 1] = make_double2(dr, di);
      if (col == 1) {
        double2 *cn = cb + (long)((r0 + 1) & 1) * n;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const int i = s * 64 + lane;
          if (i >= 1 && i < m) cn[i - 1] = a[s];
        }
      }
    }
  }
  if (blockIdx.x == 0) {
    if (k >= 0)
      for (int i = tid; i < m; i += 64 * kSW) A[(long)k * lda + r0 + i] = vs[i];
    if (!last) {
      for (int i = tid; i + 1 < m; i += 64 * kSW) vb[(long)(r0 & 1) * n + i] = cs[1 + i];
      if (tid == 0) {
        d[r0] = cs[0].x;
        e[r0] = beta1;
        tau[r0] = t1;
      }
    }
  }
}

}  // namespace

hipError_t launch_chol(double2 *S, long ld, int n, int *info, double *scr, bool wide,
                       hipStream_t s) {
  if (n < 1 || n > kEMaxN) return hipErrorInvalidValue;
  if (n <= kEigRegN) return launch_chol_reg(S, ld, n, info, s);
  if (!wide && n <= kCholMaxN) {
    hipLaunchKernelGGL(chol_kernel, dim3(1), dim3(kET), 0, s, S, ld, n, info);
    return hipGetLastError();
  }
  double2 *w = reinterpret_cast<double2 *>(scr);
  for (int jb = 0; jb < n; jb += kCB) {
    const int mt = max(0, n - jb - kCB);
    const int t = (mt + kCT - 1) / kCT;
    hipLaunchKernelGGL(cholp_kernel, dim3(max(1, t * (t + 1) / 2)), dim3(256), 0, s, S, ld, n, jb,
                       w, info);
  }
  return hipGetLastError();
}

hipError_t launch_trsm(int mode, const double2 *T, long ldt, int n, const double2 *B, long ldb,
                       int ncol, double2 *X, long ldx, hipStream_t s) {
  if (n < 1 || n > kEMaxN || ncol < 1) return hipErrorInvalidValue;
  if (n <= 256) return launch_trsm_small(mode, T, ldt, n, B, ldb, ncol, X, ldx, s);
  const dim3 grid((ncol + 3) / 4);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, T, ldt, n, B, ldb, ncol, X, ldx);
  };
  if (n <= 512) {
    if (mode == 0) go(trsm_kernel<0, 8>);
    else if (mode == 1) go(trsm_kernel<1, 8>);
    else go(trsm_kernel<2, 8>);
  } else if (n <= 1024) {
    if (mode == 0) go(trsm_kernel<0, 16>);
    else if (mode == 1) go(trsm_kernel<1, 16>);
    else go(trsm_kernel<2, 16>);
  } else {
    if (mode == 0) go(trsm_kernel<0, 32>);
    else if (mode == 1) go(trsm_kernel<1, 32>);
    else go(trsm_kernel<2, 32>);
  }
  return hipGetLastError();
}

hipError_t launch_tridiag(double2 *A, long lda, int n, double *tri, double *scr,
                          const int *info_chol, bool wide, hipStream_t s) {
  if (n < 1 || n > kEMaxN) return hipErrorInvalidValue;
  double *d = tri, *e = tri + n;
  double2 *tau = reinterpret_cast<double2 *>(tri + 2 * n);
  if (!wide && n > kTailN && n <= kET) {   // (its row x column-group layout needs n <= kET)
    hipLaunchKernelGGL(tridiag_kernel, dim3(1), dim3(kET), 0, s, A, lda, n, d, e, tau, info_chol);
    return hipGetLastError();
  }
  const int k0 = n > kTailN ? n - kTailN : 0;   // steps taken by the step kernel
  if (k0 > 0) {
    double2 *w = reinterpret_cast<double2 *>(scr);
    for (int k = -1; k < k0; ++k) {
      const int m = n - k - 1;
      const dim3 grid((m + kSW - 1) / kSW), blk(64 * kSW);
      const int last = k == k0 - 1 ? 1 : 0;
      if (n <= 512)
        hipLaunchKernelGGL(tdstep_kernel<8>, grid, blk, 0, s, A, lda, n, k, last, d, e, tau, w,
                           info_chol);
      else if (n <= 1024)
        hipLaunchKernelGGL(tdstep_kernel<16>, grid, blk, 0, s, A, lda, n, k, last, d, e, tau, w,
                           info_chol);
      else
        hipLaunchKernelGGL(tdstep_kernel<32>, grid, blk, 0, s, A, lda, n, k, last, d, e, tau, w,
                           info_chol);
    }
  }
  return launch_tridiag_reg(A + k0 + (long)k0 * lda, lda, n - k0, d + k0, e + k0, tau + k0,
                            info_chol, s);
}

hipError_t launch_backtr(const double2 *A, long lda, int n, const double *tri, const double *Zt,
                         int ldz, int nb, double2 *Zc, long ldc, const int *info_chol,
                         const int *info_eig, hipStream_t s) {
  if (n < 1 || n > kEMaxN || nb < 1) return hipErrorInvalidValue;
  if (n <= 256)
    return launch_backtr_small(A, lda, n, tri, Zt, ldz, nb, Zc, ldc, info_chol, info_eig, s);
  const dim3 grid((nb + 3) / 4);
  if (n <= 512)
    hipLaunchKernelGGL(backtr_kernel<8>, grid, dim3(256), 0, s, A, lda, n, tri, Zt, ldz, nb, Zc,
                       ldc, info_chol, info_eig);
  else if (n <= 1024)
    hipLaunchKernelGGL(backtr_kernel<16>, grid, dim3(256), 0, s, A, lda, n, tri, Zt, ldz, nb, Zc,
                       ldc, info_chol, info_eig);
  else
    hipLaunchKernelGGL(backtr_kernel<32>, grid, dim3(256), 0, s, A, lda, n, tri, Zt, ldz, nb, Zc,
                       ldc, info_chol, info_eig);
  return hipGetLastError();
}

}  // namespace qeh
