// The subspace solver's kernels for small orders: triangular solves and
// back-transformation with two or four register slots a lane (orders up to 128
// and 256; the eight of the larger instance cost four and two times the
// instructions), Cholesky factorisation and Householder tridiagonalisation for
// orders up to 128 (the reduced problems of most served cells, and
// the last 128 orders of larger ones): one workgroup with the whole matrix in
// its registers.
//
// W waves; wave w holds columns w + W c (c < KC), lane l rows l (and l + 64):
// 4 waves of 8, 12 or 16 columns for orders up to 32, 48 and 64, 8 waves of 10 to
// 16 columns with two rows a lane up to 80, 96, 112 and 128 (256 KB of the CU's
// 512 KB register file).  A step moves vectors only through LDS.  What bounds them is the
// issue of a step's instructions and its chain, so: few waves (what each does
// for itself is paid fewer times), no branches but four stages of the step loop
// that leave out the columns (and rows) already done, and the wave that owns the
// next column brings that one up to date first and works out its pivot or
// reflector while the others still update theirs.
// Tridiagonalisation, order 48 71 us, 64 102, 80 182, 96 223, 112 279, 128 325 (at
// about 110, 43 launches of a step each and an LDS-resident last 64 took 433, at
// 64 the latter 188; 16 columns a wave whatever the order: 48 84, 80 255, 96 283).
// Cholesky: 29, 41, 58, 71, 88, 98 us (at about 110, seven launches 123).
#include "eigh_vec.h"

namespace qeh {
namespace {

// sqrt(x) and 1 / sqrt(x), x > 0: the hardware's estimate and two coupled Newton
// (Goldschmidt) steps, each with a last correction by its residual; the
// library's square root and quotient take about twice the chain.
struct Root {
  double r, inv;
};
__device__ __forceinline__ Root root_of(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double d = fma(-h, g, 0.5);
    g = fma(g, d, g);
    h = fma(h, d, h);
  }
  g = fma(fma(-g, g, x), h, g);
  h = 2.0 * h;
  return {g, fma(fma(-g, h, 1.0), h, h)};
}

// row r (wave-uniform) of a column held as rows lane and lane + 64
template <int RS> __device__ __forceinline__ double2 row_of(const double2 (&c)[RS], int r) {
  if (RS == 1 || r < 64) return lane_read(c[0], r);
  return lane_read(c[RS - 1], r - 64);
}

// Matrix columns into registers, rows [0, n) of columns [0, n); LOWER: rows >=
// column only.
template <int RS, int W, int KC, bool LOWER>
__device__ __forceinline__ void load_cols(const double2 *A, long lda, int n, int lane, int w,
                                          double2 (&a)[KC][RS]) {
#pragma unroll
  for (int c = 0; c < KC; ++c)
#pragma unroll
    for (int r = 0; r < RS; ++r) {
      const int j = w + W * c, i = lane + 64 * r;
      a[c][r] = make_double2(0.0, 0.0);
      if (j < n && i < n && (!LOWER || i >= j)) a[c][r] = A[i + (long)j * lda];
    }
}

// Steps k of [C0 W, (C0 + 4) W): columns below C0 are done, and with two rows a
// lane also rows 0 .. 63 once C0 W >= 64.
constexpr int kStage = 4;
template <int C0, int KC, typename F> __device__ __forceinline__ bool stages(F &f) {
  if constexpr (C0 >= KC) {
    return true;
  } else {
    if (!f.template stage<C0>()) return false;
    return stages<C0 + kStage, KC>(f);
  }
}

// S = L L^H in place (lower triangle read and written); info = 0, or j + 1 if
// the leading (j + 1) x (j + 1) minor is not positive definite (L incomplete).
// Right-looking, one column and one barrier a step.
template <int RS, int W, int KC> struct Chol {
  double2 a[KC][RS];
  double2 *S, (*ls)[64 * RS];
  int *bad;
  long ld;
  int n, lane, w, fail;

  __device__ __forceinline__ void pivot(const double2 (&col)[RS], int k) {   // L(:, k)
    const double dk = row_of<RS>(col, k).x;
    const bool ok = dk > 0.0 && isfinite(dk);
    const Root q = root_of(ok ? dk : 1.0);
#pragma unroll
    for (int r = 0; r < RS; ++r) {
      const int i = lane + 64 * r;
      double2 l = cscale(col[r], q.inv);
      if (i <= k) l = make_double2(i == k ? q.r : 0.0, 0.0);
      ls[k & 1][i] = l;
      if (ok && i >= k && i < n) S[i + (long)k * ld] = l;
    }
    if (lane == 0) bad[k & 1] = ok ? 0 : 1;
  }
  template <int C0> __device__ __forceinline__ bool stage() {
    constexpr int R0 = C0 * W >= 64 ? RS - 1 : 0;
    const int end = min(n, (C0 + kStage) * W);
    for (int k = C0 * W; k < end; ++k) {
      __syncthreads();
      const double2 *l = ls[k & 1];
      if (bad[k & 1]) {   // uniform
        fail = k + 1;
        return false;
      }
      double2 lr[RS];
#pragma unroll
      for (int r = R0; r < RS; ++r) lr[r] = l[lane + 64 * r];
      if (((k + 1) & (W - 1)) == w && k + 1 < n) {   // its owner: the next column first
        double2 col[RS];
#pragma unroll
        for (int c = C0; c < KC && c <= C0 + kStage; ++c)
          if (w + W * c == k + 1)
#pragma unroll
            for (int r = 0; r < RS; ++r) col[r] = a[c][r];
        const double2 lj = row_of<RS>(lr, k + 1);
#pragma unroll
        for (int r = R0; r < RS; ++r) col[r] = csub(col[r], cmulc(lr[r], lj));
        pivot(col, k + 1);
      }
#pragma unroll
      for (int c = C0; c < KC; ++c) {
        const double2 lj = l[w + W * c];
#pragma unroll
        for (int r = R0; r < RS; ++r) a[c][r] = csub(a[c][r], cmulc(lr[r], lj));
      }
    }
    return true;
  }
};

template <int RS, int W, int KC>
__global__ __launch_bounds__(64 * W) void chol_reg_kernel(double2 *S, long ld, int n, int *info) {
  __shared__ double2 ls[2][64 * RS];
  __shared__ int bad[2];
  Chol<RS, W, KC> t;
  t.S = S;
  t.ls = ls;
  t.bad = bad;
  t.ld = ld;
  t.n = n;
  t.lane = threadIdx.x & 63;
  t.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  t.fail = 0;
  load_cols<RS, W, KC, true>(S, ld, n, t.lane, t.w, t.a);
  if (t.w == 0) t.pivot(t.a[0], 0);
  stages<0, KC>(t);
  if (threadIdx.x == 0) *info = t.fail;
}

// A (m x m Hermitian, full storage) = Q T Q^H: d, e, tau and the reflectors
// (column k: v_k in rows k + 1.., v_k[k + 1] = 1) as the step kernels leave
// them.  Step k: y = A22 v, a column's entry by the wave that holds it (A22 is
// Hermitian: y_j is the column's conjugate times v); w = t y + alpha v with
// alpha = -1/2 |t|^2 (v^H y), which is real, in every wave; A22 -= v w^H + w v^H,
// the next column first, whose owner then forms the next reflector.
template <int RS, int W, int KC> struct Tridiag {
  double2 a[KC][RS];
  double2 *A, (*vs)[64 * RS], *ys, *ts, *tau;
  double *d, *e;
  long lda;
  int m, lane, w;

  // v_k and t_k from the updated column k
  __device__ __forceinline__ void reflect(const double2 (&col)[RS], int k) {
    double2 alpha = row_of<RS>(col, k + 1);
    const double dk = row_of<RS>(col, k).x;
    auto norm2 = [&](double up) {   // of rows > k + 1, scaled by up
      double sq = 0.0;
#pragma unroll
      for (int r = 0; r < RS; ++r)   // (rows >= m hold zeros)
        if (lane + 64 * r > k + 1) {
          const double2 z = cscale(col[r], up);
          sq += z.x * z.x + z.y * z.y;
        }
      return wave_sum(sq);
    };
    double up = 1.0, xn2 = norm2(up), n2 = alpha.x * alpha.x + alpha.y * alpha.y + xn2;
    if (n2 < 0x1p-900) {   // uniform; the squares would lose their digits
      up = 0x1p500;
      alpha = cscale(alpha, up);
      xn2 = norm2(up);
      n2 = alpha.x * alpha.x + alpha.y * alpha.y + xn2;
    }
    double beta = alpha.x;
    double2 t = make_double2(0.0, 0.0), scale = make_double2(0.0, 0.0);
    if (xn2 != 0.0 || alpha.y != 0.0) {   // uniform
      const Root q = root_of(n2);
      beta = -copysign(q.r, alpha.x);
      const double2 ab = make_double2(alpha.x - beta, alpha.y);
      const double den = ab.x * ab.x + ab.y * ab.y;
      t = make_double2(quot(-ab.x, beta), quot(-ab.y, beta));
      scale = make_double2(up * quot(ab.x, den), -up * quot(ab.y, den));   // 1 / (alpha - beta)
    }
#pragma unroll
    for (int r = 0; r < RS; ++r) {
      const int i = lane + 64 * r;
      double2 v = cmul(col[r], scale);
      if (i <= k + 1) v = make_double2(i == k + 1 ? 1.0 : 0.0, 0.0);
      vs[k & 1][i] = v;
      if (i > k && i < m) A[i + (long)k * lda] = v;   // (only its owner reads a column)
    }
    if (lane == 0) {
      ts[k & 1] = t;
      d[k] = dk;
      e[k] = beta / up;
      tau[k] = t;
    }
  }
  template <int C0> __device__ __forceinline__ bool stage() {
    constexpr int R0 = C0 * W >= 64 ? RS - 1 : 0;
    constexpr int NC = KC - C0 > 8 ? 16 : KC - C0 > 4 ? 8 : 4;   // columns in the lane sums
    constexpr int CB = KC - NC;   // (below 0: zeros fill up the first values)
    const int end = min(m - 1, (C0 + kStage) * W);
    for (int k = C0 * W; k < end; ++k) {
      __syncthreads();
      const double2 t = ts[k & 1], *vk = vs[k & 1];
      const bool refl = t.x != 0.0 || t.y != 0.0;   // uniform
      double2 v[RS], wv[RS];
#pragma unroll
      for (int r = 0; r < RS; ++r) wv[r] = make_double2(0.0, 0.0);
#pragma unroll
      for (int r = R0; r < RS; ++r) v[r] = vk[lane + 64 * r];
      if (refl) {
        double x[2 * NC];
#pragma unroll
        for (int c = CB; c < KC; ++c) {
          double2 y = make_double2(0.0, 0.0);
          if (c >= C0) {
            y = cmulc(v[R0], a[c][R0]);
            if (R0 + 1 < RS) y = cadd(y, cmulc(v[RS - 1], a[c][RS - 1]));
          }
          x[2 * (c - CB)] = y.x;
          x[2 * (c - CB) + 1] = y.y;
        }
        const double ysum = LaneSums<2 * NC, 32>::of(x, lane);
        constexpr int LV = 32 / NC;   // lanes per value
        if ((lane & (LV - 1)) == 0 && (CB >= 0 || CB + lane / (2 * LV) >= 0))
          reinterpret_cast<double *>(ys)[2 * (w + W * (CB + lane / (2 * LV))) +
                                         ((lane / LV) & 1)] = ysum;
        __syncthreads();
        double2 yv[RS];
        double s = 0.0;
#pragma unroll
        for (int r = R0; r < RS; ++r) {   // rows <= k: v is zero, w is kept zero
          const int i = lane + 64 * r;
          yv[r] = i > k && i < W * KC ? ys[i] : make_double2(0.0, 0.0);
          s += yv[r].x * v[r].x + yv[r].y * v[r].y;
        }
        const double al = -0.5 * (t.x * t.x + t.y * t.y) * wave_sum(s);
#pragma unroll
        for (int r = R0; r < RS; ++r) wv[r] = cadd(cmul(t, yv[r]), cscale(v[r], al));
      }
      if (((k + 1) & (W - 1)) == w) {   // its owner: the next column first
        double2 col[RS];
#pragma unroll
        for (int c = C0; c < KC && c <= C0 + kStage; ++c)
          if (w + W * c == k + 1)
#pragma unroll
            for (int r = 0; r < RS; ++r) col[r] = a[c][r];
        if (refl) {
          const double2 vj = row_of<RS>(v, k + 1), wj = row_of<RS>(wv, k + 1);
#pragma unroll
          for (int r = R0; r < RS; ++r)
            col[r] = csub(col[r], cadd(cmulc(v[r], wj), cmulc(wv[r], vj)));
        }
        if (k + 2 < m) {
          reflect(col, k + 1);
        } else {
          const double dm = row_of<RS>(col, k + 1).x;
          if (lane == 0) d[k + 1] = dm;
        }
      }
      if (refl) {
#pragma unroll
        for (int c = C0; c < KC; ++c) {
          const double2 vj = vk[w + W * c], wj = lane_read(wv[W * c / 64], (w + W * c) & 63);
#pragma unroll
          for (int r = R0; r < RS; ++r)
            a[c][r] = csub(a[c][r], cadd(cmulc(v[r], wj), cmulc(wv[r], vj)));
        }
      }
    }
    return true;
  }
};

template <int RS, int W, int KC>
__global__ __launch_bounds__(64 * W) void tridiag_reg_kernel(double2 *A, long lda, int m,
                                                             double *d, double *e, double2 *tau,
                                                             const int *info_chol) {
  if (*info_chol != 0) return;
  __shared__ double2 vs[2][64 * RS], ys[64 * RS], ts[2];
  Tridiag<RS, W, KC> t;
  t.A = A;
  t.vs = vs;
  t.ys = ys;
  t.ts = ts;
  t.tau = tau;
  t.d = d;
  t.e = e;
  t.lda = lda;
  t.m = m;
  t.lane = threadIdx.x & 63;
  t.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_cols<RS, W, KC, false>(A, lda, m, t.lane, t.w, t.a);
  if (t.w == 0 && m > 1) t.reflect(t.a[0], 0);
  stages<0, KC>(t);
  if (m == 1 && threadIdx.x == 0) d[0] = t.a[0][0].x;
}

}  // namespace

hipError_t launch_chol_reg(double2 *S, long ld, int n, int *info, hipStream_t s) {
  if (n < 1 || n > kEigRegN) return hipErrorInvalidValue;
  auto go = [&](auto kern, int waves) {
    hipLaunchKernelGGL(kern, dim3(1), dim3(64 * waves), 0, s, S, ld, n, info);
    return hipGetLastError();
  };
  return n <= 32   ? go(chol_reg_kernel<1, 4, 8>, 4)
         : n <= 48 ? go(chol_reg_kernel<1, 4, 12>, 4)
         : n <= 64 ? go(chol_reg_kernel<1, 4, 16>, 4)
         : n <= 80 ? go(chol_reg_kernel<2, 8, 10>, 8)
         : n <= 96 ? go(chol_reg_kernel<2, 8, 12>, 8)
         : n <= 112 ? go(chol_reg_kernel<2, 8, 14>, 8)
                     : go(chol_reg_kernel<2, 8, 16>, 8);
}

hipError_t launch_tridiag_reg(double2 *A, long lda, int m, double *d, double *e, double2 *tau,
                              const int *info_chol, hipStream_t s) {
  if (m < 1 || m > kEigRegN) return hipErrorInvalidValue;
  auto go = [&](auto kern, int waves) {
    hipLaunchKernelGGL(kern, dim3(1), dim3(64 * waves), 0, s, A, lda, m, d, e, tau, info_chol);
    return hipGetLastError();
  };
  return m <= 32   ? go(tridiag_reg_kernel<1, 4, 8>, 4)
         : m <= 48 ? go(tridiag_reg_kernel<1, 4, 12>, 4)
         : m <= 64 ? go(tridiag_reg_kernel<1, 4, 16>, 4)
         : m <= 80 ? go(tridiag_reg_kernel<2, 8, 10>, 8)
         : m <= 96 ? go(tridiag_reg_kernel<2, 8, 12>, 8)
         : m <= 112 ? go(tridiag_reg_kernel<2, 8, 14>, 8)
                     : go(tridiag_reg_kernel<2, 8, 16>, 8);
}

hipError_t launch_trsm_small(int mode, const double2 *T, long ldt, int n, const double2 *B,
                             long ldb, int ncol, double2 *X, long ldx, hipStream_t s) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((ncol + 3) / 4), dim3(256), 0, s, T, ldt, n, B, ldb, ncol, X,
                       ldx);
    return hipGetLastError();
  };
  if (n <= 128)
    return mode == 0   ? go(trsm_kernel<0, 2>)
           : mode == 1 ? go(trsm_kernel<1, 2>)
                       : go(trsm_kernel<2, 2>);
  return mode == 0   ? go(trsm_kernel<0, 4>)
         : mode == 1 ? go(trsm_kernel<1, 4>)
                     : go(trsm_kernel<2, 4>);
}

hipError_t launch_backtr_small(const double2 *A, long lda, int n, const double *tri,
                               const double *Zt, int ldz, int nb, double2 *Zc, long ldc,
                               const int *info_chol, const int *info_eig, hipStream_t s) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((nb + 3) / 4), dim3(256), 0, s, A, lda, n, tri, Zt, ldz, nb, Zc,
                       ldc, info_chol, info_eig);
    return hipGetLastError();
  };
  return n <= 128 ? go(backtr_kernel<2>) : go(backtr_kernel<4>);
}

}  // namespace qeh
