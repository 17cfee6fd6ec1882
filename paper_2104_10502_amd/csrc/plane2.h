// Plane pass with two-factor line transforms (square planes, N1 = N2 = N = A B
// with A, B <= 16): included by plane2_f32.hip and plane2_f64.hip, which
// compile it for one precision each.
//
// A line of N points is transformed in two passes over LDS, each holding one
// factor's points in a thread's registers:
//   inverse: for each b < B, DFT_A over x[a B + b];  then for each k < A, the
//     twiddles W^{b k} and DFT_B over b, giving X[k + A q], q < B;
//   forward: for each k < A, DFT_B over f[k + A q], twiddles; then for each
//     b < B, DFT_A over k, giving F[a B + b].
// Intermediate element (k, b) sits at slot k B + b.  The second inverse pass
// leaves X[k + A q] at slot k B + q and the first forward pass reads it there,
// so no pass moves data: columns leave row y = k + A q at slot k B + q, and
// for the x rows the second inverse pass, the V(r) multiply and the first
// forward pass are one pass on registers.
//
// The sphere fills the x-extent columns and about half of each line: column
// c = h - hmin and y position k - kmin (shifted from h, k mod N; the shift's
// phase in real space cancels between the two directions, V being real), so
// with at most (A + 1) / 2 values of a in use (HALF) the first inverse pass
// loads and the last forward pass stores only those.
//
// LDS holds the x-extent columns (T); a row needs N slots for its
// intermediate, of which the first k0 B (k0 = ext / B) are the row's own column
// entries and the rest lie in E, for rc rows at a time.  One workgroup: one
// z plane of one band (or Gamma band pair), ids remapped so that each XCD
// walks contiguous (plane, band) runs with the band fastest (V from its L2).
//
// Bound: vector issue (about 30 lane operations a point and transform, twice
// the 5 n log2 n count's share of the FMA rate) and, where one workgroup of
// columns fills a CU's LDS, the latency of its passes between barriers.
// Measured per launch inside H psi (kernel traces of the same card), the kernel it
// replaced (LDS passes of radix 2 to 8; * lane pairs, quads or octets with DPP
// exchanges) -> this one:
//   FP32  45^3, 202 bands            186 ->   54 us    FP64  30^3, 16    16 ->   9
//         72^3, 128 bands            176* -> 139             72^3, 128  360* -> 287
//         135^3, 32 band pairs       874 ->  296             135^3, 32 2434 ->  752
//         160 x 160 x 168, 64 pairs 1493* -> 1015
// The plane pass alone, without the matrix products before it, runs at a higher
// clock: 135^3 FP32 880 -> 263, the last line 1471* -> 822.  At half-filled lines of
// all compiled sizes (64 bands): 1.5 to 6.7 times as fast as the LDS passes, 1.0
// to 1.4 as the lane pairs (16 sizes), 1.3 to 1.5 as the quads in FP64 (10) and 1.5 to
// 1.8 as quads and octets in FP32 (5); FP64 lines above 135 points do not fit.
#pragma once

#include <algorithm>

#include "cplx.h"
#include "fft_reg.h"
#include "qeh_internal.h"

namespace qeh {
namespace plane2 {

// N = A B: the most nearly square factors, A >= B (the fused middle pass keeps
// B values and their twiddles in registers; an unequal pair measured up to a
// third slower), A <= 16 except 125 = 25 x 5.
constexpr int factor_b(int n) {
  int best = 0;
  for (int b = 2; b * b <= n; ++b)
    if (n % b == 0) best = b;
  return best;
}
// Threads per workgroup: about two of a plane's row items ((row, k) and
// (row, b)) per thread and pass at the smaller sizes; the large single-precision
// planes leave room for one workgroup per CU and take 1024 (the plane pass alone,
// N = 160, 64 band pairs of 168 planes: 822 us, 1040 with 512; 135, 32 pairs of 135:
// 263 and 327; N = 72: 256 and 512 within 1%), the FP64 ones 512 (1024 would spill).
constexpr int threads(bool f64, int n) {
  return n <= 36 ? 128
         : n <= (f64 ? 60 : 72) ? 256
         : f64 || n <= 120 || n / factor_b(n) > 16 ? 512 : 1024;
}
constexpr int pitch_b(int b) { return b | 1; }   // odd: no bank conflicts over k
constexpr int pitch(int n, int b) { return (n / b * pitch_b(b)) | 1; }
// Single-precision sizes whose columns can exceed LDS also have a form without
// that padding (TIGHT), for the extents at which the padded columns leave too
// little LDS for rows (two_geometry): its bank conflicts cost up to 3% (N = 160, 95
// columns, 64 bands of 24 planes: 181 and 187 us), more rows at a time give more back
// (113 columns 423 -> 221 us).
constexpr bool has_tight(bool f64, int n) {
  return !f64 && pitch_b(factor_b(n)) != factor_b(n) && 8 * n * pitch(n, factor_b(n)) > kLdsMax;
}

template <typename C, int N, int B, int NT, bool HALF, bool TIGHT>
__global__ __launch_bounds__(NT) void k2_two(
    C *__restrict__ sbuf, const typename real_of<C>::type *__restrict__ vs,
    const int *__restrict__ tidx, const C *__restrict__ tw, int nst, int n3, int ext, int rc,
    int nbk, int per_xcd) {
  using R = typename real_of<C>::type;
  constexpr int A = N / B, BP = TIGHT ? B : pitch_b(B), LD = TIGHT ? N | 1 : pitch(N, B);
  constexpr int AU = HALF ? (A + 1) / 2 : A;   // values of a that hold data
  constexpr int NTA = NT / A * A;              // threads of the (line, k) passes: fixed k
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int id = blockIdx.x;
  const int logical = (id & 7) * per_xcd + (id >> 3);
  if (logical >= nbk * n3) return;
  const int z = logical / nbk;
  const int b0 = logical - z * nbk;
  const int tid = threadIdx.x;
  C *T = reinterpret_cast<C *>(smem_raw);
  C *E = T + ext * LD;
  const int ER = rc | 1;
  const int k0 = ext / B;
  C *plane = sbuf + ((size_t)b0 * n3 + z) * nst;

  const int myk = tid % A;
  C w[B];   // W^{b k} = exp(-2 pi i b k / N)
#pragma unroll
  for (int b = 1; b < B; ++b) w[b] = tw[b * myk];

  for (int i = tid; i < ext * (AU * B); i += NT) {
    const int c = i / (AU * B), p = i - c * (AU * B);
    T[c * LD + p / B * BP + p % B] = cmk<C>(0, 0);
  }
  __syncthreads();
  for (int s = tid; s < nst; s += NT) T[tidx[s]] = plane[s];
  __syncthreads();

  // ---- y inverse
  for (int t = tid; t < ext * B; t += NT) {
    const int c = t / B, b = t - c * B;
    C *col = T + c * LD + b;
    C v[A];
#pragma unroll
    for (int a = 0; a < A; ++a) v[a] = a < AU ? col[a * BP] : cmk<C>(0, 0);
    regfft::Fft<C, A, true>::run(v);
#pragma unroll
    for (int k = 0; k < A; ++k) col[k * BP] = v[k];
  }
  __syncthreads();
  if (tid < NTA)
    for (int t = tid; t < ext * A; t += NTA) {
      C *col = T + t / A * LD + myk * BP;
      C v[B];
#pragma unroll
      for (int b = 0; b < B; ++b) v[b] = b ? cmulc(col[b], w[b]) : col[0];
      regfft::Fft<C, B, true>::run(v);
#pragma unroll
      for (int q = 0; q < B; ++q) col[q] = v[q];
    }
  __syncthreads();

  // ---- rows, rc at a time
  for (int s0 = 0; s0 < N; s0 += rc) {
    const int nr = min(rc, N - s0);
    for (int t = tid; t < nr * B; t += NT) {
      const int r = t / B, b = t - r * B;
      const int s = s0 + r;
      C *row = T + b * LD + s / B * BP + s % B;
      C *er = E + b * ER + r;
      C v[A];
#pragma unroll
      for (int a = 0; a < A; ++a)
        v[a] = a < AU && a * B + b < ext ? row[a * (B * LD)] : cmk<C>(0, 0);
      regfft::Fft<C, A, true>::run(v);
#pragma unroll
      for (int k = 0; k < A; ++k) {
        C *p = k < k0 ? row + k * (B * LD) : er + (k - k0) * (B * ER);
        *p = v[k];
      }
    }
    __syncthreads();
    if (tid < NTA)
      for (int t = tid; t < nr * A; t += NTA) {
        const int r = t / A;
        const int s = s0 + r;
        const int sk = s / B, sq = s - sk * B;
        const int st = myk < k0 ? LD : ER;
        C *p = myk < k0 ? T + myk * (B * LD) + sk * BP + sq : E + (myk - k0) * (B * ER) + r;
        const R *vr = vs + ((size_t)z * N + sk + A * sq) * N + myk;
        R pot[B];
#pragma unroll
        for (int q = 0; q < B; ++q) pot[q] = vr[A * q];
        C v[B];
#pragma unroll
        for (int b = 0; b < B; ++b) v[b] = b ? cmulc(p[b * st], w[b]) : p[0];
        regfft::Fft<C, B, true>::run(v);
#pragma unroll
        for (int q = 0; q < B; ++q) v[q] = cscale(v[q], pot[q]);
        regfft::Fft<C, B, false>::run(v);
#pragma unroll
        for (int b = 0; b < B; ++b) p[b * st] = b ? cmul(v[b], w[b]) : v[0];
      }
    __syncthreads();
    for (int t = tid; t < nr * B; t += NT) {
      const int r = t / B, b = t - r * B;
      const int s = s0 + r;
      C *row = T + b * LD + s / B * BP + s % B;
      const C *er = E + b * ER + r;
      C v[A];
#pragma unroll
      for (int k = 0; k < A; ++k) {
        const C *p = k < k0 ? row + k * (B * LD) : er + (k - k0) * (B * ER);
        v[k] = *p;
      }
      regfft::Fft<C, A, false>::run(v);
#pragma unroll
      for (int a = 0; a < AU; ++a)
        if (a * B + b < ext) row[a * (B * LD)] = v[a];
    }
    __syncthreads();
  }

  // ---- y forward
  if (tid < NTA)
    for (int t = tid; t < ext * A; t += NTA) {
      C *col = T + t / A * LD + myk * BP;
      C v[B];
#pragma unroll
      for (int q = 0; q < B; ++q) v[q] = col[q];
      regfft::Fft<C, B, false>::run(v);
#pragma unroll
      for (int b = 0; b < B; ++b) col[b] = b ? cmul(v[b], w[b]) : v[0];
    }
  __syncthreads();
  for (int t = tid; t < ext * B; t += NT) {
    const int c = t / B, b = t - c * B;
    C *col = T + c * LD + b;
    C v[A];
#pragma unroll
    for (int k = 0; k < A; ++k) v[k] = col[k * BP];
    regfft::Fft<C, A, false>::run(v);
#pragma unroll
    for (int a = 0; a < AU; ++a) col[a * BP] = v[a];
  }
  __syncthreads();
  for (int s = tid; s < nst; s += NT) plane[s] = T[tidx[s]];
}

template <typename C, int N> hipError_t launch(const qeh_ctx *c, int nbk) {
  using R = typename real_of<C>::type;
  constexpr int B = factor_b(N), NT = threads(sizeof(R) == 8, N);
  const int total = nbk * c->n3, per_xcd = (total + 7) / 8;
  auto go = [&](auto kern) {
    if (c->two.lds > 64 * 1024)
      (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)c->two.lds);
    hipLaunchKernelGGL(kern, dim3(8 * per_xcd), dim3(NT), c->two.lds, c->stream,
                       reinterpret_cast<C *>(c->d.sbuf), reinterpret_cast<const R *>(c->d.vs),
                       c->d.tidx2, reinterpret_cast<const C *>(c->d.tw) + c->tw_off[0], c->nst,
                       c->n3, c->ext, c->two.rc, nbk, per_xcd);
    return hipGetLastError();
  };
  if constexpr (has_tight(sizeof(R) == 8, N))
    if (c->two.tight)
      return c->two.half ? go(&k2_two<C, N, B, NT, true, true>)
                         : go(&k2_two<C, N, B, NT, false, true>);
  return c->two.half ? go(&k2_two<C, N, B, NT, true, false>)
                     : go(&k2_two<C, N, B, NT, false, false>);
}

// Charge density: one workgroup = one z plane of one subgroup of bands, the
// inverse half of the plane pass for one band after another.  The last pass
// holds each point's f_b |psi_b|^2 sums in registers, in band order: a thread
// meets the same (row, k) items for every band (NCH chunks of RC rows, unrolled;
// the y and x shifts are unit-modulus phases of psi).  Bound: as the plane pass.
// 72^3, FP64, 128 bands: 266 us on lane quads -> 184.  Whole density of 64 bands
// on lane quads (FP64) or pairs, or separate column and row passes (*) -> this
// kernel (us):
//   FP64  45^3 172* -> 66   60^3 131 -> 96   80^3 423* -> 172   120^2 x 48 519* -> 251
//   FP32  45^3 151* -> 65   60^3  92 -> 80   80^3 184 -> 115    120^2 x 48 328* -> 202
// Threads: the sums leave no room for more than 512, and in FP64 up to N = 96 two
// workgroups of 256 beat one of 512 (N = 72: 182 and 203 us).
constexpr int density_threads(bool f64, int n) {
  const int t = threads(f64, n), cap = f64 && n <= 96 ? 256 : 512;
  return t < cap ? t : cap;
}
// Row chunks: so few that two workgroups (or, where the columns alone fill half a
// CU's LDS, one) are resident with the sphere filling half of a line; 0: not
// compiled (too many registers: more than four chunks, 64 sums a thread, A > 16).
constexpr int density_chunks(bool f64, int n) {
  const int b = factor_b(n), a = n / b, cs = f64 ? 16 : 8;
  const int ext = n / 2 + 1, tile = ext * pitch(n, b) * cs, row = (a - ext / b) * b * cs;
  const int cap = tile < 72 * 1024 ? 80 * 1024 : 156 * 1024;
  const int nta = density_threads(f64, n) / a * a;
  for (int c = 1; c <= 4 && a <= 16; ++c) {
    const int rc = (n + c - 1) / c;
    if (tile + (rc | 1) * row <= cap) return c * ((rc * a + nta - 1) / nta) * b <= 64 ? c : 0;
  }
  return 0;
}

template <typename C, int N, int NCH, bool HALF>
__global__ __launch_bounds__(density_threads(sizeof(C) == 16, N)) void k2d_two(
    const C *__restrict__ sbuf, const double *__restrict__ occ, double *__restrict__ partial,
    const int *__restrict__ tidx, const C *__restrict__ tw, int nst, int n3, int ext, int nbk,
    int bsub) {
  constexpr int NT = density_threads(sizeof(C) == 16, N);
  constexpr int B = factor_b(N), A = N / B, BP = pitch_b(B), LD = pitch(N, B);
  constexpr int AU = HALF ? (A + 1) / 2 : A;
  constexpr int NTA = NT / A * A;
  constexpr int RC = (N + NCH - 1) / NCH, ER = RC | 1, IT = (RC * A + NTA - 1) / NTA;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int z = blockIdx.x % n3, sub = blockIdx.x / n3;
  const int tid = threadIdx.x;
  C *T = reinterpret_cast<C *>(smem_raw);
  C *E = T + ext * LD;
  const int k0 = ext / B;
  const int myk = tid % A;
  C w[B];   // W^{b k} = exp(-2 pi i b k / N)
#pragma unroll
  for (int b = 1; b < B; ++b) w[b] = tw[b * myk];
  double acc[NCH][IT][B];
#pragma unroll
  for (int i = 0; i < NCH * IT * B; ++i) acc[i / (IT * B)][i / B % IT][i % B] = 0.0;

  for (int band = sub * bsub; band < min(nbk, (sub + 1) * bsub); ++band) {
    const C *plane = sbuf + ((size_t)band * n3 + z) * nst;
    for (int i = tid; i < ext * (AU * B); i += NT) {
      const int c = i / (AU * B), p = i - c * (AU * B);
      T[c * LD + p / B * BP + p % B] = cmk<C>(0, 0);
    }
    __syncthreads();
    for (int s = tid; s < nst; s += NT) T[tidx[s]] = plane[s];
    __syncthreads();
    for (int t = tid; t < ext * B; t += NT) {
      const int c = t / B, b = t - c * B;
      C *col = T + c * LD + b;
      C v[A];
#pragma unroll
      for (int a = 0; a < A; ++a) v[a] = a < AU ? col[a * BP] : cmk<C>(0, 0);
      regfft::Fft<C, A, true>::run(v);
#pragma unroll
      for (int k = 0; k < A; ++k) col[k * BP] = v[k];
    }
    __syncthreads();
    if (tid < NTA)
      for (int t = tid; t < ext * A; t += NTA) {
        C *col = T + t / A * LD + myk * BP;
        C v[B];
#pragma unroll
        for (int b = 0; b < B; ++b) v[b] = b ? cmulc(col[b], w[b]) : col[0];
        regfft::Fft<C, B, true>::run(v);
#pragma unroll
        for (int q = 0; q < B; ++q) col[q] = v[q];
      }
    __syncthreads();
    const double f = occ[band];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int s0 = ch * RC, nr = min(RC, N - s0);
      for (int t = tid; t < nr * B; t += NT) {
        const int r = t / B, b = t - r * B;
        const int s = s0 + r;
        C *row = T + b * LD + s / B * BP + s % B;
        C *er = E + b * ER + r;
        C v[A];
#pragma unroll
        for (int a = 0; a < A; ++a)
          v[a] = a < AU && a * B + b < ext ? row[a * (B * LD)] : cmk<C>(0, 0);
        regfft::Fft<C, A, true>::run(v);
#pragma unroll
        for (int k = 0; k < A; ++k) {
          C *p = k < k0 ? row + k * (B * LD) : er + (k - k0) * (B * ER);
          *p = v[k];
        }
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int t = tid + it * NTA;
        if (tid < NTA && t < nr * A) {
          const int r = t / A, s = s0 + r;
          const int st = myk < k0 ? LD : ER;
          const C *p =
              myk < k0 ? T + myk * (B * LD) + s / B * BP + s % B : E + (myk - k0) * (B * ER) + r;
          C v[B];
#pragma unroll
          for (int b = 0; b < B; ++b) v[b] = b ? cmulc(p[b * st], w[b]) : p[0];
          regfft::Fft<C, B, true>::run(v);
#pragma unroll
          for (int q = 0; q < B; ++q) {
            const double re = v[q].x, im = v[q].y;
            acc[ch][it][q] += f * (re * re + im * im);
          }
        }
      }
      __syncthreads();
    }
  }
  double *out = partial + ((size_t)sub * n3 + z) * N * N;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int t = tid + it * NTA, s = ch * RC + t / A;
      if (tid < NTA && t < min(RC, N - ch * RC) * A) {
        double *row = out + (size_t)(s / B + A * (s % B)) * N + myk;
#pragma unroll
        for (int q = 0; q < B; ++q) row[A * q] = acc[ch][it][q];
      }
    }
}

// LDS of the density pass, 0 where it is not compiled.
template <typename C, int N> size_t density_lds(int ext) {
  constexpr int NCH = density_chunks(sizeof(C) == 16, N);
  if constexpr (NCH == 0) {
    return 0;
  } else {
    constexpr int B = factor_b(N), A = N / B, RC = (N + NCH - 1) / NCH;
    return sizeof(C) * ((size_t)ext * pitch(N, B) + (size_t)(A - ext / B) * B * (RC | 1));
  }
}

template <typename C, int N>
hipError_t launch_density(const qeh_ctx *c, int nbk, int bsub, const double *occ,
                          double *partial) {
  constexpr int NCH = density_chunks(sizeof(C) == 16, N);
  if constexpr (NCH == 0) {
    return hipErrorInvalidValue;
  } else {
    const size_t lds = density_lds<C, N>(c->ext);
    const int nsub = (nbk + bsub - 1) / bsub;
    auto go = [&](auto kern) {
      if (lds > 64 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      hipLaunchKernelGGL(kern, dim3((unsigned)nsub * c->n3),
                         dim3(density_threads(sizeof(C) == 16, N)), lds, c->stream,
                         reinterpret_cast<const C *>(c->d.sbuf), occ, partial, c->d.tidx2,
                         reinterpret_cast<const C *>(c->d.tw) + c->tw_off[0], c->nst, c->n3, c->ext,
                         nbk, bsub);
      return hipGetLastError();
    };
    return c->two.half ? go(&k2d_two<C, N, NCH, true>) : go(&k2d_two<C, N, NCH, false>);
  }
}

// The 49 sizes compiled: products of 2, 3, 5, 7 up to 192 with both factors <= 16,
// without 49 and 98, and 125.
#define QEH_TWO_SIZES(X)                                                                       \
  X(12) X(14) X(15) X(16) X(18) X(20) X(21) X(24) X(25) X(27) X(28) X(30) X(32) X(35) X(36)    \
  X(40) X(42) X(45) X(48) X(50) X(54) X(56) X(60) X(63) X(64) X(70) X(72) X(75) X(80) X(81)    \
  X(84) X(90) X(96) X(100) X(105) X(108) X(112) X(120) X(125) X(126) X(128) X(135) X(140)      \
  X(144) X(150) X(160) X(168) X(180) X(192)

}  // namespace plane2
}  // namespace qeh
