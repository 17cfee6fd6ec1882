// Triangular solves and the back-transformation of the subspace solver: one wave
// per column, its entries in register slots (included by eigh_small.hip for
// orders up to 256 and by eigh_kernels.hip for larger ones).
#pragma once

#include "eigh_common.h"

namespace qeh {
namespace {

// ---------------------------------------------------------------- triangular solves
// One wave per right-hand side column j; the column's n <= 64 NS entries sit in
// registers (row s * 64 + lane in slot s).
//   MODE 0: L x = b,   L lower (T), b = B(:, j)
//   MODE 1: L x = b,   b = conj(M(j, :)) with M = B (column j of M^H)
//   MODE 2: U x = b,   U upper (T), b = B(:, j)   (backward)
// The diagonal of T is real (a Cholesky factor).
//
// By blocks of 64 rows (one slot): the diagonal block of T is staged in LDS
// (shared by the workgroup's four waves), its columns divided by their diagonal
// entries and zero outside the triangle, so that a step is a scalar read of one
// unknown and an update of all lanes; the quotient by the diagonal follows at
// the end.  The slots on the far side then take the block's contribution,
// x_s -= T_sb x_b, from L2.  Both run eight columns at a time with the next
// eight columns' reads in flight.  Each x_i still receives its terms T_ik x_k
// in the order of k.  Orders around 120: 14 us (31 with a branch and the quotient
// on the chain of each step).
// One block round: solve block (= slot) B, then the far side.  B is a
// template argument so that every slot index is a compile-time constant and
// x stays in registers.
template <int MODE, int B, int NS>
__device__ __forceinline__ void trsm_round(double2 (&x)[NS], const double2 *__restrict__ T,
                                           long ldt, int n, int lane, double2 (*Tb)[64],
                                           double *rd) {
  constexpr int U = 8;
  const int nbk = (n + 63) / 64;
  if (B >= nbk) return;   // uniform
  const int b0 = B * 64, bs = min(64, n - b0);
  const int wid = threadIdx.x >> 6;
  double2 st[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int c = wid + 4 * u;
    st[u] = make_double2(0.0, 0.0);
    if (lane < bs && c < bs && (MODE == 2 ? lane < c : lane > c))
      st[u] = T[(b0 + lane) + (long)(b0 + c) * ldt];
  }
  __syncthreads();   // the previous round's block is no longer read
  if ((int)threadIdx.x < 64)
    rd[threadIdx.x] =
        (int)threadIdx.x < bs
            ? 1.0 / T[(b0 + threadIdx.x) + (long)(b0 + threadIdx.x) * ldt].x
            : 0.0;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 16; ++u) Tb[wid + 4 * u][lane] = cscale(st[u], rd[wid + 4 * u]);
  __syncthreads();
  double2 tv[U], tn[U];
  // the block's unknowns (columns bs .. 63 are zero)
  const int ng = (bs + U - 1) / U;
  auto grp = [&](int g) { return (MODE == 2 ? ng - 1 - g : g) * U; };
#pragma unroll
  for (int u = 0; u < U; ++u) tn[u] = Tb[grp(0) + u][lane];
  for (int g = 0; g < ng; ++g) {
    const int c0 = grp(g);
#pragma unroll
    for (int u = 0; u < U; ++u) tv[u] = tn[u];
    if (g + 1 < ng) {
#pragma unroll
      for (int u = 0; u < U; ++u) tn[u] = Tb[grp(g + 1) + u][lane];
    }
#pragma unroll
    for (int v = 0; v < U; ++v) {
      const int u = MODE == 2 ? U - 1 - v : v;
      x[B] = csub(x[B], cmul(tv[u], lane_read(x[B], c0 + u)));
    }
  }
  x[B] = cscale(x[B], rd[lane]);
  // the far side: x_s -= T(rows of s, columns of B) x_B
#pragma unroll
  for (int s2 = 0; s2 < NS; ++s2) {
    const bool far = MODE == 2 ? s2 < B : s2 > B;
    const int i = s2 * 64 + lane;
    if (far && s2 < nbk) {
      const double2 *tc = T + min(i, n - 1) + (long)b0 * ldt;
      double2 acc = x[s2];
      auto fetch = [&](int c0) {   // (columns past the block: x_B is zero there)
#pragma unroll
        for (int u = 0; u < U; ++u) tn[u] = tc[(long)min(c0 + u, bs - 1) * ldt];
      };
      fetch(0);
      for (int c0 = 0; c0 < bs; c0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) tv[u] = tn[u];
        if (c0 + U < bs) fetch(c0 + U);
#pragma unroll
        for (int u = 0; u < U; ++u) acc = csub(acc, cmul(tv[u], lane_read(x[B], c0 + u)));
      }
      if (i < n) x[s2] = acc;
    }
  }
}

// All block rounds, in solve order (forward for MODE 0 / 1, backward for 2).
template <int MODE, int NS, int Q>
__device__ __forceinline__ void trsm_rounds(double2 (&x)[NS], const double2 *__restrict__ T,
                                            long ldt, int n, int lane, double2 (*Tb)[64],
                                            double *rd) {
  if constexpr (Q < NS) {
    trsm_round<MODE, MODE == 2 ? NS - 1 - Q : Q, NS>(x, T, ldt, n, lane, Tb, rd);
    trsm_rounds<MODE, NS, Q + 1>(x, T, ldt, n, lane, Tb, rd);
  }
}

// NS register slots per lane (orders up to 64 NS).
template <int MODE, int NS>
__global__ __launch_bounds__(256) void trsm_kernel(const double2 *__restrict__ T, long ldt, int n,
                                                   const double2 *__restrict__ B, long ldb,
                                                   int ncol, double2 *__restrict__ X, long ldx) {
  __shared__ double2 Tb[64][64];   // diagonal block: Tb[c][r] = T(b0 + r, b0 + c) rd[c]
  __shared__ double rd[64];        // reciprocals of its diagonal
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  const bool live = j < ncol;   // every wave stays for the barriers
  double2 x[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = s * 64 + lane;
    double2 v = make_double2(0.0, 0.0);
    if (live && i < n) {
      if (MODE == 1) {
        const double2 m = B[j + (long)i * ldb];
        v = make_double2(m.x, -m.y);
      } else {
        v = B[i + (long)j * ldb];
      }
    }
    x[s] = v;
  }
  trsm_rounds<MODE, NS, 0>(x, T, ldt, n, lane, Tb, rd);
  if (!live) return;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = s * 64 + lane;
    if (i < n) X[i + (long)j * ldx] = x[s];
  }
}

// ---------------------------------------------------------------- back-transformation
constexpr int kTK = 8;   // reflectors staged per chunk

// Zc(:, j) = Q Zt(:, j) = H_0 (H_1 ( ... H_{n-2} Zt(:, j))), one wave per
// column; the four waves of a workgroup share the reflectors, staged through
// LDS kTK at a time with the next chunk's loads in flight.  Two reflectors at
// a time: with a = v^H z, b = u^H z and g = u^H v from one pass over the lanes,
// H_u H_v z = z - c v - d u, c = t_v a, d = t_u (b - c g).  Orders around 120,
// 64 columns: 24 us (57 one at a time with two separate sums each, 110 with
// eight register slots a lane).
template <int NS>   // register slots per lane: orders up to 64 NS
__global__ __launch_bounds__(256) void backtr_kernel(const double2 *__restrict__ A, long lda, int n,
                                                     const double *__restrict__ tri,
                                                     const double *__restrict__ Zt, int ldz,
                                                     int nb, double2 *__restrict__ Zc, long ldc,
                                                     const int *info_chol, const int *info_eig) {
  if (*info_chol != 0 || *info_eig != 0) return;
  constexpr int TK = NS <= 16 ? kTK : 2;   // reflectors per chunk (LDS, registers)
  constexpr int R = NS * 64;
  __shared__ double2 Vs[TK][R];
  __shared__ double2 ts[TK];
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  const bool live = j < nb;   // every wave stays for the barriers
  const double2 *tau = reinterpret_cast<const double2 *>(tri + 2 * n);
  double2 z[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = s * 64 + lane;
    z[s] = make_double2(live && i < n ? Zt[i + (long)j * ldz] : 0.0, 0.0);
  }
  // reflectors k = kl .. kh (rows > k; zeros elsewhere, and past kh) in
  // descending chunks, the next chunk's loads in flight during the current
  // one's reflectors
  constexpr int NPF = TK * R / 256;
  double2 pf[NPF], pt = make_double2(0.0, 0.0);
  auto fetch = [&](int kh) {
    const int kl = max(0, kh - TK + 1);
#pragma unroll
    for (int u = 0; u < NPF; ++u) {
      const int idx = threadIdx.x + u * 256;
      const int k = kl + idx / R, i = idx % R;
      pf[u] = make_double2(0.0, 0.0);
      if (k <= kh && i > k && i < n) pf[u] = A[i + (long)k * lda];
    }
    if (threadIdx.x < TK) {
      const int k = kl + threadIdx.x;
      pt = make_double2(0.0, 0.0);
      if (k <= kh) pt = tau[k];
    }
  };
  const int top = n - 2;
  if (top >= 0) fetch(top);
  for (int kh = top; kh >= 0; kh -= TK) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NPF; ++u) {
      const int idx = threadIdx.x + u * 256;
      Vs[idx / R][idx % R] = pf[u];
    }
    if (threadIdx.x < TK) ts[threadIdx.x] = pt;
    __syncthreads();
    if (kh - TK >= 0) fetch(kh - TK);
#pragma unroll 1
    for (int q = TK - 2; q >= 0; q -= 2) {
      const double2 *v = Vs[q + 1], *u = Vs[q];   // v first
      double x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = 0.0;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const double2 vi = v[s * 64 + lane], ui = u[s * 64 + lane], zi = z[s];
        x[0] += vi.x * zi.x + vi.y * zi.y;
        x[1] += vi.x * zi.y - vi.y * zi.x;
        x[2] += ui.x * zi.x + ui.y * zi.y;
        x[3] += ui.x * zi.y - ui.y * zi.x;
        x[4] += ui.x * vi.x + ui.y * vi.y;
        x[5] += ui.x * vi.y - ui.y * vi.x;
      }
      const double y = LaneSums<8, 32>::of(x, lane);
      const double2 a = make_double2(lane_read(y, 0), lane_read(y, 8)),
                    b = make_double2(lane_read(y, 16), lane_read(y, 24)),
                    g = make_double2(lane_read(y, 32), lane_read(y, 40));
      const double2 c = cmul(ts[q + 1], a), d = cmul(ts[q], csub(b, cmul(c, g)));
#pragma unroll
      for (int s = 0; s < NS; ++s)
        z[s] = csub(z[s], cadd(cmul(c, v[s * 64 + lane]), cmul(d, u[s * 64 + lane])));
    }
  }
  if (!live) return;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int i = s * 64 + lane;
    if (i < n) Zc[i + (long)j * ldc] = z[s];
  }
}

}  // namespace
}  // namespace qeh
