// FP64 complex matrix products on the MFMA units, and the D scaling of the
// projector coefficients (the single-precision products: split_gemm.hip).
//
// Uses: the pseudopotential contribution of H (becp = beta^H psi, ps = D becp,
// hpsi += beta ps), which the paper lists among the ported Hamiltonian
// kernels, and the Rayleigh-Ritz reductions / Ritz rotations of the Davidson
// solver, which the paper runs through GPU BLAS (section "Evolution of the
// GPU-enabled version").
//
// A complex product is three real MFMA products on planar (re, im) tiles
// (Gauss's three-multiplication form):
//   P1 += Ar Br,   P2 += Ai Bi,   P3 += (Ar + Ai)(Br + Bi),
//   Cr = P1 - P2,  Ci = P3 - P1 - P2.
// The operand sums are formed in registers after the LDS reads.  The form is
// normwise stable; its rounding error is a small constant multiple of that of
// the four-product form (Cr = Ar Br - Ai Bi, Ci = Ar Bi + Ai Br), and it issues
// a quarter fewer MFMAs.  The kernels are held to three waves per SIMD (the
// third accumulator set would otherwise push them to two).
// Two cheaper forms serve the Gamma-point projections (RM = 1: only the real
// part of C is wanted, Cr = P1 - P2; RM = 2: A is real, Cr = sum Ar Br and
// Ci = sum Ar Bi): two MFMA products per step instead of three.
// WGM x WGN waves (64 * WGM * WGN threads); each wave owns a
// (BM/WGM) x (BN/WGN) block of C built from 16 x 16 x 4 MFMA tiles.  Long K is
// split into fixed chunks whose partial results are summed in double by a
// separate kernel in a fixed order (deterministic, no atomics).
#include <algorithm>

#include "cplx.h"
#include "qeh_internal.h"

namespace qeh {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void mfma(double a, double b, doublex4 &c) {
  c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// One workgroup: a BM x BN tile of C over the K slice [kbeg, kend).  Global
// tiles are prefetched into registers while the MFMAs consume the LDS copy of
// the previous slice (two LDS buffers, one barrier per slice).
template <int BMODE, int BM, int BN, int BK, int RM, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(3)))
void cgemm_kernel(
    const double2 *__restrict__ A, long lda, const double2 *__restrict__ B, long ldb,
    double2 *__restrict__ C, long ldc, int M, int N, int K, int conjA, int conjB, int accumulate,
    int kchunk, long split_stride, int tiles_m, int tiles_n, int ntiles, int per_xcd) {
  constexpr int kGT = 64 * WGM * WGN;
  constexpr int BKP = BK + 1;
  constexpr int TM = BM / (16 * WGM);
  constexpr int TN = BN / (16 * WGN);
  constexpr int NA = BM * BK / kGT;
  constexpr int NB = BN * BK / kGT;
  static_assert(TM * 16 * WGM == BM && TN * 16 * WGN == BN && BK % 4 == 0, "tile / wave mismatch");
  static_assert(NA * kGT == BM * BK && NB * kGT == BN * BK, "tile / thread mismatch");
  __shared__ double As[2][2][BM * BKP];   // [buffer][re, im]
  __shared__ double Bs[2][2][BN * BKP];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm0 = (wave / WGN) * (BM / WGM);
  const int wn0 = (wave % WGN) * (BN / WGN);
  // Workgroup ids are dealt round-robin to the 8 XCDs (each with its own L2);
  // the remap gives each XCD a contiguous run of (m tile fastest, n tile,
  // K slice), so tiles that read the same operand rows run on one XCD
  // back to back.
  const int id = blockIdx.x;
  const int logical = (id & 7) * per_xcd + (id >> 3);
  if (logical >= ntiles) return;
  const int mt = logical % tiles_m;
  const int nt = (logical / tiles_m) % tiles_n;
  const int kz = logical / (tiles_m * tiles_n);
  const int m0 = mt * BM;
  const int n0 = nt * BN;
  const int kbeg = kz * kchunk;
  const int kend = min(K, kbeg + kchunk);
  double2 *Cz = C + (long)kz * split_stride;
  const double sa = conjA ? -1.0 : 1.0;
  const double sb = conjB ? -1.0 : 1.0;

  doublex4 p1[TM][TN], p2[TM][TN], p3[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p1[i][j][e] = 0.0;
        p2[i][j][e] = 0.0;
        p3[i][j][e] = 0.0;
      }

  // Global operand loads for one K slice into registers.
  auto gload = [&](int k0, double2 *ra, double2 *rb) {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int e = tid + u * kGT;
      const int r = e / BK, k = e % BK;
      const int gm = m0 + r, gk = k0 + k;
      ra[u] = (gm < M && gk < kend) ? A[(long)gm * lda + gk] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int e = tid + u * kGT;
      const int k = BMODE == 0 ? e % BK : e / BN;
      const int r = BMODE == 0 ? e / BK : e % BN;
      const int gn = n0 + r, gk = k0 + k;
      const long at = BMODE == 0 ? (long)gn * ldb + gk : (long)gk * ldb + gn;
      rb[u] = (gn < N && gk < kend) ? B[at] : make_double2(0.0, 0.0);
    }
  };
  auto sstore = [&](int buf, const double2 *ra, const double2 *rb) {
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int e = tid + u * kGT;
      const int r = e / BK, k = e % BK;
      As[buf][0][r * BKP + k] = ra[u].x;
      As[buf][1][r * BKP + k] = sa * ra[u].y;
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int e = tid + u * kGT;
      const int k = BMODE == 0 ? e % BK : e / BN;
      const int r = BMODE == 0 ? e / BK : e % BN;
      Bs[buf][0][r * BKP + k] = rb[u].x;
      Bs[buf][1][r * BKP + k] = sb * rb[u].y;
    }
  };

  const int lr = lane % 16;   // row (A) / column (B) inside a block
  const int lk = lane / 16;   // k inside a step of 4

  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      double ar[TM], ai[TM], as[TM], br[TN], bi[TN], bs[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int off = (wm0 + i * 16 + lr) * BKP + kk + lk;
        ar[i] = As[buf][0][off];
        ai[i] = As[buf][1][off];
        as[i] = ar[i] + ai[i];
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int off = (wn0 + j * 16 + lr) * BKP + kk + lk;
        br[j] = Bs[buf][0][off];
        bi[j] = Bs[buf][1][off];
        bs[j] = br[j] + bi[j];
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          mfma(ar[i], br[j], p1[i][j]);
          if (RM == 2) {
            mfma(ar[i], bi[j], p2[i][j]);
          } else {
            mfma(ai[i], bi[j], p2[i][j]);
            if (RM == 0) mfma(as[i], bs[j], p3[i][j]);
          }
        }
    }
  };

  // one slice in flight: loaded during the MFMAs of the previous one
  double2 ra[NA], rb[NB];
  if (kbeg < kend) {
    gload(kbeg, ra, rb);
    sstore(0, ra, rb);
  }
  __syncthreads();
  int buf = 0;
  for (int k0 = kbeg; k0 < kend; k0 += BK) {
    const bool more = k0 + BK < kend;
    if (more) gload(k0 + BK, ra, rb);
    compute(buf);
    if (more) sstore(buf ^ 1, ra, rb);
    __syncthreads();
    buf ^= 1;
  }

  // ---- epilogue.  Column lane%16 of each block; accumulator entry r holds
  // row lane/16+4*r (the f32 instructions lay out D differently).
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gm = m0 + wm0 + i * 16 + lk + 4 * r;
        const int gn = n0 + wn0 + j * 16 + lr;
        if (gm < M && gn < N) {
          double2 *p = Cz + (long)gm * ldc + gn;
          double cr = RM == 2 ? p1[i][j][r] : p1[i][j][r] - p2[i][j][r];
          double ci = RM == 0   ? p3[i][j][r] - p1[i][j][r] - p2[i][j][r]
                      : RM == 2 ? p2[i][j][r]
                                : 0.0;
          if (accumulate) {
            const double2 v = *p;
            cr += v.x;
            ci += v.y;
          }
          *p = make_double2(cr, ci);
        }
      }
}

// 64 x 64 tiles on four waves, K slices of 8.
template <int BMODE, int RM> hipError_t run_tile(const GemmDesc &g, hipStream_t s) {
  constexpr int BM = 64, BN = 64;
  const int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
  const long total = (long)tm * tn * g.nsplit;
  if (total > (1L << 30)) return hipErrorInvalidValue;
  const int per_xcd = (int)((total + 7) / 8);
  const int kchunk = g.nsplit > 1 ? g.kchunk : g.K;
  hipLaunchKernelGGL((cgemm_kernel<BMODE, BM, BN, 8, RM, 2, 2>), dim3(8 * per_xcd), dim3(256), 0,
                     s, reinterpret_cast<const double2 *>(g.A), g.lda,
                     reinterpret_cast<const double2 *>(g.B), g.ldb,
                     reinterpret_cast<double2 *>(g.C), g.ldc, g.M, g.N, g.K, g.conjA, g.conjB,
                     g.accumulate, kchunk, g.split_stride, tm, tn, (int)total, per_xcd);
  return hipGetLastError();
}

template <typename TP, typename TC>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const TP *__restrict__ part,
                                                            long stride, int nsplit, int M, int N,
                                                            long ldp, TC *__restrict__ C, long ldc,
                                                            int accumulate) {
  const long total = (long)M * N;
  for (long t = blockIdx.x * (long)blockDim.x + threadIdx.x; t < total;
       t += (long)gridDim.x * blockDim.x) {
    const int m = (int)(t / N), n = (int)(t % N);
    const TP *pp = part + (long)m * ldp + n;
    double sr = 0.0, si = 0.0;
    int s = 0;
    for (; s + 8 <= nsplit; s += 8) {   // split order kept; 8 loads in flight
      TP v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = pp[(long)(s + u) * stride];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        sr += static_cast<double>(v[u].x);
        si += static_cast<double>(v[u].y);
      }
    }
    for (; s < nsplit; ++s) {
      const TP v = pp[(long)s * stride];
      sr += static_cast<double>(v.x);
      si += static_cast<double>(v.y);
    }
    TC *p = C + (long)m * ldc + n;
    if (accumulate) {
      sr += static_cast<double>(p->x);
      si += static_cast<double>(p->y);
    }
    TC o;
    o.x = static_cast<typename real_of<TC>::type>(sr);
    o.y = static_cast<typename real_of<TC>::type>(si);
    *p = o;
  }
}

// ---------------------------------------------------------------- D scaling
// grid (chunk, band).  Chunk c covers whole atoms [p0, p1), p1 - p0 <= 256.
// Gamma contexts (gpsi set): the partials sum conj(beta) psi over the stored
// half sphere, and the full-sphere projection is real:
//   becp = 2 Re(sum) - beta(0) psi(0)   (G = 0 counted once; beta(0) real).
__device__ __forceinline__ void store_ps(double2 *ps, long i, double sr, double si) {
  ps[i] = make_double2(sr, si);
}
__device__ __forceinline__ void store_ps(float2 *ps, long i, double sr, double si) {
  ps[i] = make_float2((float)sr, (float)si);
}
// Gamma, single precision: ps is real, stored as one float per entry
__device__ __forceinline__ void store_ps(float *ps, long i, double sr, double) {
  ps[i] = (float)sr;
}

template <typename TP, typename TS>
__global__ __launch_bounds__(256) void dscale_kernel(
    const TP *__restrict__ part, long split_stride, int nsplit, int nkb, TS *__restrict__ ps,
    const double2 *__restrict__ dmat, const int *__restrict__ pj0, const int *__restrict__ pnb,
    const int *__restrict__ pdoff, const int *__restrict__ chunk,
    const double2 *__restrict__ gpsi, long ldpsi, const TP *__restrict__ gbeta, long ldb) {
  __shared__ double2 becp[256];
  const int p0 = chunk[blockIdx.x], p1 = chunk[blockIdx.x + 1];
  const int b = blockIdx.y;
  const int t = threadIdx.x;
  const int j = p0 + t;
  if (j < p1) {
    // partials summed in split order; loads issued eight at a time so that
    // several are in flight per thread
    const TP *pp = part + (long)b * nkb + j;
    double sr = 0.0, si = 0.0;
    int s = 0;
    for (; s + 8 <= nsplit; s += 8) {
      TP v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = pp[(long)(s + u) * split_stride];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        sr += static_cast<double>(v[u].x);
        si += static_cast<double>(v[u].y);
      }
    }
    for (; s < nsplit; ++s) {
      const TP v = pp[(long)s * split_stride];
      sr += static_cast<double>(v.x);
      si += static_cast<double>(v.y);
    }
    if (gpsi) {
      const double p0 = gpsi[(long)b * ldpsi].x;
      const double b0 = static_cast<double>(gbeta[(long)j * ldb].x);
      sr = 2.0 * sr - b0 * p0;
      si = 0.0;
    }
    becp[t] = make_double2(sr, si);
  }
  __syncthreads();
  if (j < p1) {
    const int j0 = pj0[j], nbk = pnb[j];
    const double2 *drow = dmat + pdoff[j];
    double sr = 0.0, si = 0.0;
    for (int q = 0; q < nbk; ++q) {
      const double2 d = drow[q];
      const double2 v = becp[j0 + q - p0];
      sr += d.x * v.x - d.y * v.y;
      si += d.x * v.y + d.y * v.x;
    }
    store_ps(ps, (long)b * nkb + j, sr, si);
  }
}

}  // namespace

// The Gamma-point forms: RM = 1 for beta^H psi (bmode 0), RM = 2 for beta ps
// (bmode 1, A = ps real in complex storage).
hipError_t launch_cgemm(const GemmDesc &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipSuccess;
  if (g.ta != T_D2 || g.tb != T_D2 || g.tc != T_D2) return hipErrorInvalidValue;
  if (g.rmode == 0) return g.bmode == 0 ? run_tile<0, 0>(g, s) : run_tile<1, 0>(g, s);
  if (g.rmode == 1 && g.bmode == 0) return run_tile<0, 1>(g, s);
  if (g.rmode == 2 && g.bmode == 1) return run_tile<1, 2>(g, s);
  return hipErrorInvalidValue;
}

hipError_t launch_splitk_reduce(const void *part, int tp, long stride, int nsplit, int M, int N,
                                long ldp, double2 *C, long ldc, int accumulate, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const long total = (long)M * N;
  const int blocks = (int)std::min<long>((total + 255) / 256, 4096);
  if (tp == T_D2)
    hipLaunchKernelGGL((splitk_reduce_kernel<double2, double2>), dim3(blocks), dim3(256), 0, s,
                       reinterpret_cast<const double2 *>(part), stride, nsplit, M, N, ldp, C, ldc,
                       accumulate);
  else
    hipLaunchKernelGGL((splitk_reduce_kernel<float2, double2>), dim3(blocks), dim3(256), 0, s,
                       reinterpret_cast<const float2 *>(part), stride, nsplit, M, N, ldp, C, ldc,
                       accumulate);
  return hipGetLastError();
}

hipError_t launch_dscale(const qeh_ctx *c, int nbk, const double2 *psi, long ldpsi,
                         const double2 *mat) {
  if (c->nkb == 0) return hipSuccess;
  if (!mat) mat = c->d.dmat;
  dim3 grid(c->nchunk, nbk);
  const long ss = (long)c->block * c->nkb;
  const double2 *gpsi = c->gamma ? psi : nullptr;
  if (c->prec == QEH_FP64) {
    hipLaunchKernelGGL((dscale_kernel<double2, double2>), grid, dim3(256), 0, c->stream,
                       reinterpret_cast<const double2 *>(c->d.part), ss, c->nsplit, c->nkb,
                       reinterpret_cast<double2 *>(c->d.ps), mat, c->d.pj0, c->d.pnb,
                       c->d.pdoff, c->d.chunk, gpsi, ldpsi,
                       reinterpret_cast<const double2 *>(c->d.beta), (long)c->ldb);
  } else if (c->gamma) {
    // real ps, one float per entry: half the A operand of the beta ps product
    hipLaunchKernelGGL((dscale_kernel<float2, float>), grid, dim3(256), 0, c->stream,
                       reinterpret_cast<const float2 *>(c->d.part), ss, c->nsplit, c->nkb,
                       reinterpret_cast<float *>(c->d.ps), mat, c->d.pj0, c->d.pnb,
                       c->d.pdoff, c->d.chunk, gpsi, ldpsi,
                       reinterpret_cast<const float2 *>(c->d.beta), (long)c->ldb);
  } else {
    hipLaunchKernelGGL((dscale_kernel<float2, float2>), grid, dim3(256), 0, c->stream,
                       reinterpret_cast<const float2 *>(c->d.part), ss, c->nsplit, c->nkb,
                       reinterpret_cast<float2 *>(c->d.ps), mat, c->d.pj0, c->d.pnb,
                       c->d.pdoff, c->d.chunk, gpsi, ldpsi,
                       reinterpret_cast<const float2 *>(c->d.beta), (long)c->ldb);
  }
  return hipGetLastError();
}

}  // namespace qeh
