// z transforms of the sticks with two-factor lines (N3 = A B): K1 (sphere ->
// sticks -> inverse z) and K3 (forward z -> sphere), included by
// stick2_f32.hip and stick2_f64.hip, which compile it for one precision each.
//
// A workgroup takes S consecutive sticks of one band: their sphere runs are one
// contiguous range of psi (lexicographic Miller order).  A line is transformed
// in two passes as in the plane kernel: K1 places the coefficients in their line
// in LDS, runs DFT_A per (stick, b) in LDS and DFT_B per (stick, k) straight to
// the plane-major stick buffer; K3 is its mirror image.  Lanes run over sticks,
// so the buffer's rows of consecutive sticks are read and written whole, and a
// line goes through LDS once between its two passes.  The sphere fills about a
// quarter of a line at either end: only the values a < AL and a >= A - AH are
// cleared, loaded by the first K1 pass and stored by the last K3 pass (HALF).
//
// Bound: HBM (psi, the stick buffer, H psi: 684 MB for K1 of the last line by the
// counters, 3.9 TB/s; a copy reaches 4.9).
// Measured, LDS passes of radix 2 to 8 (* lane pairs; Gamma: with the kernel
// that separated K3's pairs) -> this kernel, K1, K3 (us; kernel traces of H psi):
//   FP64  30, 16 bands          7.9,   9.1 ->   4.0,   3.7
//         72, 128 bands        57.8,  66.4 ->  40.4,  46.2
//         135, 32 Gamma pairs   118,   155 ->    78,    88
//   FP32  45, 202 bands        17.9,  18.1 ->  13.1,  13.5
//         72, 128 bands *      32.7,  36.7 ->  33.2,  33.1
//         135, 32 Gamma pairs  92.9,   125 ->    63,    63
//         168, 64 Gamma pairs   206,   336 ->   176,   164
// (K1 of 72 points alone is as fast as it was on lane pairs.)
#pragma once

#include <algorithm>

#include "cplx.h"
#include "fft_reg.h"
#include "plane2.h"
#include "qeh_internal.h"

namespace qeh {
namespace stick2 {

using plane2::factor_b;
using plane2::pitch;
using plane2::pitch_b;

constexpr int kThreads = 256;
constexpr int low_values(int a) { return a / 4 + 1; }    // values of a with l >= 0
constexpr int high_values(int a) { return (a + 3) / 4; } // and with l < 0 (HALF)

// The z lines of one workgroup in LDS: 2^sl of them, and the twiddles.
template <typename C, int N, bool HALF> struct Lines {
  static constexpr int B = factor_b(N), A = N / B, BP = pitch_b(B), LD = pitch(N, B);
  static constexpr int AL = HALF ? low_values(A) : A, AH = HALF ? high_values(A) : 0;
  C *tile, *twl;
  int sl, tid, nt;

  __device__ __forceinline__ Lines(void *smem, int sl_)
      : tile(static_cast<C *>(smem) + N), twl(static_cast<C *>(smem)), sl(sl_), tid(threadIdx.x),
        nt(blockDim.x) {}
  static __device__ __forceinline__ bool used(int a) { return a < AL || a >= A - AH; }
  __device__ __forceinline__ void twiddles(const C *__restrict__ tw) {
    for (int i = tid; i < N; i += nt) twl[i] = tw[i];
  }
  __device__ __forceinline__ void clear() {
    for (int i = tid; i < (AL + AH) * B << sl; i += nt) {
      const int s = i & ((1 << sl) - 1), p = i >> sl;
      tile[s * LD + (p / B < AL ? p / B : p / B + A - AL - AH) * BP + p % B] = cmk<C>(0, 0);
    }
  }
  // put(s, z, value): line s (it decides which are live)
  template <typename F> __device__ __forceinline__ void inverse(F put) {
    for (int t = tid; t < B << sl; t += nt) {
      C *line = tile + (t & ((1 << sl) - 1)) * LD + (t >> sl);
      C v[A];
#pragma unroll
      for (int a = 0; a < A; ++a) v[a] = used(a) ? line[a * BP] : cmk<C>(0, 0);
      regfft::Fft<C, A, true>::run(v);
#pragma unroll
      for (int k = 0; k < A; ++k) line[k * BP] = v[k];
    }
    __syncthreads();
    for (int t = tid; t < A << sl; t += nt) {
      const int s = t & ((1 << sl) - 1), k = t >> sl;
      const C *line = tile + s * LD + k * BP;
      C v[B];
#pragma unroll
      for (int b = 0; b < B; ++b) v[b] = b ? cmulc(line[b], twl[b * k]) : line[0];
      regfft::Fft<C, B, true>::run(v);
      put(s, k, v);
    }
  }
  // get(s, k, v): v[q] = plane k + A q of line s; false for a line that is not live
  template <typename F> __device__ __forceinline__ void forward(F get) {
    for (int t = tid; t < A << sl; t += nt) {
      const int s = t & ((1 << sl) - 1), k = t >> sl;
      C v[B];
      if (!get(s, k, v)) continue;
      C *line = tile + s * LD + k * BP;
      regfft::Fft<C, B, false>::run(v);
#pragma unroll
      for (int b = 0; b < B; ++b) line[b] = b ? cmul(v[b], twl[b * k]) : v[0];
    }
    __syncthreads();
    for (int t = tid; t < B << sl; t += nt) {
      C *line = tile + (t & ((1 << sl) - 1)) * LD + (t >> sl);
      C v[A];
#pragma unroll
      for (int k = 0; k < A; ++k) v[k] = line[k * BP];
      regfft::Fft<C, A, false>::run(v);
#pragma unroll
      for (int a = 0; a < A; ++a)
        if (used(a)) line[a * BP] = v[a];
    }
    __syncthreads();
  }
};

// The sticks of a workgroup.  Complex: lines 0 .. 2^sl - 1 are sticks s0 ...
// Gamma: half of the lines are consecutive sticks from u0 of the upper half of
// the sphere (from the middle stick h = k = 0 up), the other half their mirror
// images, so that a stored coefficient, which stands for G and -G, is read (and
// H psi written) once; the middle stick is its own mirror image and takes both
// in its upper line.
template <int LD> struct Sticks {
  int s0, u0, m0, mid, nst, hs;   // hs: lines per half (Gamma), m0: stick of line hs
  __device__ __forceinline__ Sticks(bool gam, int sl, int nst_) : nst(nst_) {
    hs = gam ? 1 << (sl - 1) : 1 << sl;
    mid = (nst - 1) / 2;
    s0 = blockIdx.x << sl;
    u0 = gam ? mid + blockIdx.x * hs : s0;
    m0 = nst - u0 - hs;
  }
  // stick of a line, or -1
  __device__ __forceinline__ int of(int line) const {
    const int s = line < hs ? u0 + line : m0 + line - hs;
    return line < hs ? (s < nst ? s : -1) : (s >= 0 && s < mid ? s : -1);
  }
  __device__ __forceinline__ int upper(int gm) const { return gm - u0 * LD; }
  __device__ __forceinline__ int lower(int gm) const { return gm - (m0 - hs) * LD; }
};

// psi32: the block's single-precision copy (rows of ld32), or null.  Gamma:
// launch "band" b is the pair (2b, 2b + 1) of nbk bands, or pairs[b], as
// psi_a + i psi_b over the full sphere (Im psi(0) is not referenced).
template <typename C, int N, bool HALF, bool GAM>
__global__ __launch_bounds__(kThreads) void k1_two(
    const double2 *__restrict__ psi, int ldpsi, C *__restrict__ sbuf,
    const int *__restrict__ stick_off, const int *__restrict__ gmap, const C *__restrict__ tw,
    int nst, int sl, float2 *__restrict__ psi32, int ld32, int nbk, int nh,
    const int2 *__restrict__ pairs) {
  using L = Lines<C, N, HALF>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  L ln(smem_raw, sl);
  const Sticks<L::LD> st(GAM, sl, nst);
  const int b0 = blockIdx.y;
  ln.twiddles(tw);
  ln.clear();
  __syncthreads();
  const int ue = min(st.u0 + st.hs, nst);
  if constexpr (!GAM) {
    const double2 *pb = psi + (size_t)b0 * ldpsi;
    for (int g = stick_off[st.u0] + ln.tid, g1 = stick_off[ue]; g < g1; g += ln.nt) {
      const double2 v = pb[g];
      ln.tile[st.upper(gmap[g])] = ccast<C>(v);
      if (psi32) psi32[(size_t)b0 * ld32 + g] = make_float2((float)v.x, (float)v.y);
    }
  } else {
    const int2 rows = pairs ? pairs[b0] : make_int2(2 * b0, 2 * b0 + 1 < nbk ? 2 * b0 + 1 : -1);
    const double2 *pa = psi + (size_t)rows.x * ldpsi, *pb = psi + (size_t)rows.y * ldpsi;
    const int z = nh - 1, gm = stick_off[st.mid];
    for (int h = max(stick_off[st.u0] - z, 0) + ln.tid, h1 = stick_off[ue] - z; h < h1;
         h += ln.nt) {
      double2 va = pa[h], vb = make_double2(0.0, 0.0);
      if (rows.y >= 0) vb = pb[h];
      if (psi32) {
        psi32[(size_t)rows.x * ld32 + h] = make_float2((float)va.x, (float)va.y);
        if (rows.y >= 0)
          psi32[(size_t)rows.y * ld32 + h] = make_float2((float)vb.x, (float)vb.y);
      }
      if (h == 0) va.y = vb.y = 0.0;
      ln.tile[st.upper(gmap[z + h])] = ccast<C>(make_double2(va.x - vb.y, va.y + vb.x));
      if (h > 0) {
        const int q = gmap[z - h];
        ln.tile[z - h >= gm ? st.upper(q) : st.lower(q)] =
            ccast<C>(make_double2(va.x + vb.y, vb.x - va.y));
      }
    }
  }
  __syncthreads();
  C *out = sbuf + (size_t)b0 * N * nst;
  ln.inverse([&](int line, int k, const C(&v)[L::B]) {
    const int s = st.of(line);
    if (s < 0) return;
#pragma unroll
    for (int q = 0; q < L::B; ++q) out[(size_t)(k + L::A * q) * nst + s] = v[q];
  });
}

// H psi over the sphere with the kinetic term.  Gamma (pair b: bands 2b, 2b + 1
// of nbk): from C = F(V psi_a) + i F(V psi_b), F(V psi_a)(G) = (C(G) +
// conj C(-G)) / 2 and F(V psi_b)(G) = (C(G) - conj C(-G)) / (2i).
template <typename C, int N, bool HALF, bool GAM>
__global__ __launch_bounds__(kThreads) void k3_two(
    const C *__restrict__ sbuf, const double2 *__restrict__ psi, int ldpsi,
    double2 *__restrict__ hpsi, int ldh, const double *__restrict__ kin,
    const int *__restrict__ stick_off, const int *__restrict__ gmap, const C *__restrict__ tw,
    int nst, int sl, int nbk, int nh) {
  using L = Lines<C, N, HALF>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  L ln(smem_raw, sl);
  const Sticks<L::LD> st(GAM, sl, nst);
  const int b0 = blockIdx.y;
  ln.twiddles(tw);
  __syncthreads();
  const C *in = sbuf + (size_t)b0 * N * nst;
  ln.forward([&](int line, int k, C(&v)[L::B]) {
    const int s = st.of(line);
    if (s < 0) return false;
#pragma unroll
    for (int q = 0; q < L::B; ++q) v[q] = in[(size_t)(k + L::A * q) * nst + s];
    return true;
  });
  const int ue = min(st.u0 + st.hs, nst);
  if constexpr (!GAM) {
    const double2 *pb = psi + (size_t)b0 * ldpsi;
    double2 *hb = hpsi + (size_t)b0 * ldh;
    for (int g = stick_off[st.u0] + ln.tid, g1 = stick_off[ue]; g < g1; g += ln.nt) {
      const double2 r = ccast<double2>(ln.tile[st.upper(gmap[g])]);
      const double2 p = pb[g];
      const double k = kin[g];
      hb[g] = make_double2(r.x + k * p.x, r.y + k * p.y);
    }
  } else {
    const double2 *pa = psi + (size_t)(2 * b0) * ldpsi;
    double2 *ha = hpsi + (size_t)(2 * b0) * ldh;
    const bool two = 2 * b0 + 1 < nbk;
    const int z = nh - 1, gm = stick_off[st.mid];
    for (int h = max(stick_off[st.u0] - z, 0) + ln.tid, h1 = stick_off[ue] - z; h < h1;
         h += ln.nt) {
      const int q = gmap[z - h];
      const double2 cp = ccast<double2>(ln.tile[st.upper(gmap[z + h])]);
      const double2 cm = ccast<double2>(ln.tile[z - h >= gm ? st.upper(q) : st.lower(q)]);
      const double k = kin[h];
      double2 va = pa[h];
      if (h == 0) va.y = 0.0;
      ha[h] = make_double2(0.5 * (cp.x + cm.x) + k * va.x, 0.5 * (cp.y - cm.y) + k * va.y);
      if (two) {
        double2 vb = pa[ldpsi + h];
        if (h == 0) vb.y = 0.0;
        ha[ldh + h] =
            make_double2(0.5 * (cp.y + cm.y) + k * vb.x, -0.5 * (cp.x - cm.x) + k * vb.y);
      }
    }
  }
}

// workgroups over the sticks (Gamma: over the upper half's)
inline unsigned groups(const qeh_ctx *c) {
  const int n = c->gamma ? (c->nst + 1) / 2 : c->nst;
  const int per = c->gamma ? 1 << (c->st2.sl - 1) : 1 << c->st2.sl;
  return (unsigned)((n + per - 1) / per);
}

template <typename C, int N>
hipError_t launch_k1(const qeh_ctx *c, int np, const double2 *psi, int ldpsi, int nbk,
                     const int2 *pairs, float2 *p32) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(groups(c), np),
                       dim3(kThreads), c->st2.lds, c->stream, psi, ldpsi,
                       reinterpret_cast<C *>(c->d.sbuf), c->d.stick_off, c->d.gmap,
                       reinterpret_cast<const C *>(c->d.tw) + c->tw_off[2], c->nst, c->st2.sl, p32,
                       c->ldb, nbk, c->npw, pairs);
    return hipGetLastError();
  };
  if (c->gamma) return c->st2.half ? go(&k1_two<C, N, true, true>) : go(&k1_two<C, N, false, true>);
  return c->st2.half ? go(&k1_two<C, N, true, false>) : go(&k1_two<C, N, false, false>);
}

template <typename C, int N>
hipError_t launch_k3(const qeh_ctx *c, int nbk, const double2 *psi, int ldpsi, double2 *hpsi,
                     int ldh) {
  const int np = c->gamma ? (nbk + 1) / 2 : nbk;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(groups(c), np),
                       dim3(kThreads), c->st2.lds, c->stream,
                       reinterpret_cast<const C *>(c->d.sbuf), psi, ldpsi, hpsi, ldh, c->d.kin,
                       c->d.stick_off, c->d.gmap,
                       reinterpret_cast<const C *>(c->d.tw) + c->tw_off[2], c->nst, c->st2.sl, nbk,
                       c->npw);
    return hipGetLastError();
  };
  if (c->gamma) return c->st2.half ? go(&k3_two<C, N, true, true>) : go(&k3_two<C, N, false, true>);
  return c->st2.half ? go(&k3_two<C, N, true, false>) : go(&k3_two<C, N, false, false>);
}

}  // namespace stick2
}  // namespace qeh
