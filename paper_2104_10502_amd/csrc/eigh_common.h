// Constants and wave / workgroup reductions of the subspace solver's kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "cplx.h"
#include "qeh_internal.h"

namespace qeh {
namespace {

constexpr int kET = 1024;            // threads of the one-workgroup kernels
constexpr int kEW = kET / 64;        // their waves
constexpr int kEMaxN = kEigMaxN;     // largest problem
constexpr double kEps = 2.220446049250313e-16;
constexpr double kTiny = 2.2250738585072014e-308;
constexpr double kDegRel = 1e-12;    // numerically equal eigenvalues (relative to ||T||)
constexpr double kCloseRel = 1e-5;   // close eigenvalues, re-orthogonalised

// a / q, 1 / q and a / q normal numbers: the hardware's estimate of 1 / q, one
// Newton step, and the quotient corrected by its remainder
__device__ __forceinline__ double quot(double a, double q) {
  double r = __builtin_amdgcn_rcp(q);
  r = fma(r, fma(-q, r, 1.0), r);
  const double y = a * r;
  return fma(fma(-q, y, a), r, y);
}

// the value of another lane of the row (DPP control word; every lane has a source)
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int CTRL> __device__ __forceinline__ double dpp_add(double v) {
  return v + dpp_mov<CTRL>(v);
}
// value of lane l (wave-uniform) of v, through the scalar unit
__device__ __forceinline__ double lane_read(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double2 lane_read(double2 v, int l) {
  return make_double2(lane_read(v.x, l), lane_read(v.y, l));
}
__device__ __forceinline__ double2 swap32(double a, double b) {   // {lower halves, upper halves}
  const long long u = __double_as_longlong(a), v = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)v, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(v >> 32), false,
                                                   false);
  return make_double2(__longlong_as_double(((long long)hi[0] << 32) | lo[0]),
                      __longlong_as_double(((long long)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double2 swap16(double a, double b) {   // {even rows, odd rows}
  const long long u = __double_as_longlong(a), v = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)v, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(v >> 32), false,
                                                   false);
  return make_double2(__longlong_as_double(((long long)hi[0] << 32) | lo[0]),
                      __longlong_as_double(((long long)hi[1] << 32) | lo[1]));
}
// Sum over the wave (all lanes active), the same value in every lane, in a
// fixed order, by exchanges between registers (a shuffle butterfly goes through
// LDS six times).
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v = dpp_add<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v = dpp_add<0x141>(v);   // row_half_mirror
  v = dpp_add<0x140>(v);   // row_mirror
  const double2 p = swap16(v, v);
  v = p.x + p.y;
  const double2 q = swap32(v, v);
  return q.x + q.y;
}

// Sums of the NV values x (a power of two) over the wave's lanes: lane l returns
// the sum of x[l / (64 / NV)].  Every exchange between lanes halves the number
// of values while there are several, so that NV values take NV - 1 + log2(64 / NV)
// additions.
template <int NV, int BIT> struct LaneSums {
  static __device__ __forceinline__ double of(const double *x, int lane) {
    constexpr int H = NV > 1 ? NV / 2 : 1;
    double y[H];
    if constexpr (BIT == 32 || BIT == 16) {
#pragma unroll
      for (int i = 0; i < H; ++i) {
        const double2 q = BIT == 32 ? swap32(x[i], x[NV > 1 ? i + H : i])
                                    : swap16(x[i], x[NV > 1 ? i + H : i]);
        y[i] = q.x + q.y;
      }
    } else {
      // row_ror:8, row_half_mirror (the lane bits below are summed later), quad_perm
      constexpr int CTRL = BIT == 8 ? 0x128 : BIT == 4 ? 0x141 : BIT == 2 ? 0x4E : 0xB1;
      if constexpr (NV > 1) {
        const bool up = (lane & BIT) != 0;
#pragma unroll
        for (int i = 0; i < H; ++i)
          y[i] = (up ? x[i + H] : x[i]) + dpp_mov<CTRL>(up ? x[i] : x[i + H]);
      } else {
        y[0] = x[0] + dpp_mov<CTRL>(x[0]);
      }
    }
    if constexpr (BIT == 1) return y[0];
    else return LaneSums<H, BIT / 2>::of(y, lane);
  }
};

// Sums over the workgroup (NW waves), identical in every thread and from run to
// run.  Two at once (red holds 2 NW doubles): the same orders as two calls of
// block_sum, one pair of barriers.
template <int NW> __device__ double2 block_sum2(double a, double b, double *red) {
  a = wave_sum(a);
  b = wave_sum(b);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = a;
    red[NW + (threadIdx.x >> 6)] = b;
  }
  __syncthreads();
  double sa = 0.0, sb = 0.0;
  for (int i = 0; i < NW; ++i) sa += red[i];
  for (int i = 0; i < NW; ++i) sb += red[NW + i];
  return make_double2(sa, sb);
}

template <int NW = kEW> __device__ double block_sum(double v, double *red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < NW; ++i) s += red[i];
  return s;
}

template <int NW> __device__ double block_max(double v, double *red) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = red[0];
  for (int i = 1; i < NW; ++i) s = fmax(s, red[i]);
  return s;
}

template <int NW> __device__ double block_min(double v, double *red) {
  return -block_max<NW>(-v, red);
}

}  // namespace
}  // namespace qeh
