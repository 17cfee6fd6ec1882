// FP64 complex matrix products on the MFMA units, and the D scaling of the
// projector coefficients (the single-precision products: split_gemm.hip).
//
// Uses: the pseudopotential contribution of H (becp = beta^H psi, ps = D becp,
// hpsi += beta ps), which the paper lists among the ported Hamiltonian
// kernels, and the Rayleigh-Ritz reductions / Ritz rotations of the Davidson
// solver, which the paper runs through GPU BLAS (section "Evolution of the
// GPU-enabled version").
//
// A complex product of the large tiles is three real MFMA products (Gauss's
// three-multiplication form, RM = 0):
//   P1 += Ar Br,   P2 += Ai Bi,   P3 += (Ar + Ai)(Br + Bi),
//   Cr = P1 - P2,  Ci = P3 - P1 - P2.
// The operand sums are formed in registers after the LDS reads.  The form is
// normwise stable; its rounding error is a small constant multiple of that of
// the four-product form (Cr = Ar Br - Ai Bi, Ci = Ar Bi + Ai Br), and it issues
// a quarter fewer MFMAs.  The kernels are held to three waves per SIMD (the
// third accumulator set would otherwise push them to two).  The flat tiles wait
// for memory rather than for the MFMAs and take the four-product form (RM = 3);
// H psi and S psi, whose bits may not depend on how the bands are grouped, take
// the form of the context's whole block in launches of any number of bands.
// Two cheaper forms serve the Gamma-point projections (RM = 1: only the real
// part of C is wanted; RM = 2: A is real, Cr = sum Ar Br and Ci = sum Ar Bi):
// two MFMA products per step.
// WGM x WGN waves (64 * WGM * WGN threads); each wave owns a
// (BM/WGM) x (BN/WGN) block of C built from 16 x 16 x 4 MFMA tiles.  Long K is
// split into fixed chunks whose partial results are summed in double by a
// separate kernel in a fixed order (deterministic, no atomics).
#include <algorithm>
#include <type_traits>

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
// the previous slice (two LDS buffers, one barrier per slice).  LDS keeps the
// elements as loaded (re, im together): one 16-byte store an element and one
// 16-byte read a fragment, free of bank conflicts at a pitch of BK + 1
// elements.  B's conjugation (CJ) is a sign in the sums.  RM = 1 and 3 add both
// products of a part into one accumulator set.
//
// Bound: the f64 matrix rate (72.7 TFLOP/s for a library product of 8192^3
// here, 62 for this kernel on 2048 x 2048 x 4096) and, at Gamma, beta from HBM
// (2.4 GB at 2048 projectors: 0.5 ms).  Planar LDS tiles with masked loads ->
// this kernel (us, kernel traces of H psi): 128 x 512, K 23 976, 199 -> 185;
// 128 x 23 976, K 512, 209 -> 195; Gamma 64 x 2 048, K 74 047, 828 -> 776;
// 64 x 74 047, K 2 048, 913 -> 837.
template <int BMODE, int BM, int BN, int BK, int RM, int WGM, int WGN, bool CJ>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(3)))
void cgemm_kernel(
    const double2 *__restrict__ A, long lda, const double2 *__restrict__ B, long ldb,
    double2 *__restrict__ C, long ldc, int M, int N, int K, int accumulate,
    int kchunk, long split_stride, int tiles_m, int tiles_n, int ntiles, int per_xcd) {
  constexpr int kGT = 64 * WGM * WGN;
  constexpr int BKP = BK + 1;
  constexpr int TM = BM / (16 * WGM);
  constexpr int TN = BN / (16 * WGN);
  constexpr int NA = BM * BK / kGT;
  constexpr int NB = BN * BK / kGT;
  static_assert(NA * kGT == BM * BK && NB * kGT == BN * BK, "tile / thread mismatch");
  __shared__ double2 As[2][BM * BKP];
  __shared__ double2 Bs[2][BN * BKP];
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
  constexpr int NP = RM == 0 ? 3 : RM >= 2 ? 2 : 1;
  doublex4 p[NP][TM][TN];
#pragma unroll
  for (int q = 0; q < NP; ++q)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) p[q][i][j][e] = 0.0;
  // Rows beyond M / N repeat the last one (their results are not stored), so
  // whole slices load without masks.
  const double2 *pa[NA], *pb[NB];
  int la[NA], lb[NB], ka[NA], kb[NB];   // LDS slot and k of each load
#pragma unroll
  for (int u = 0; u < NA; ++u) {
    const int e = tid + u * kGT;
    const int r = e / BK, k = e % BK;
    pa[u] = A + (long)min(m0 + r, M - 1) * lda + kbeg + k;
    la[u] = r * BKP + k;
    ka[u] = k;
  }
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int e = tid + u * kGT;
    const int k = BMODE == 0 ? e % BK : e / BN;
    const int r = BMODE == 0 ? e / BK : e % BN;
    const int gn = min(n0 + r, N - 1);
    pb[u] = BMODE == 0 ? B + (long)gn * ldb + kbeg + k : B + (long)(kbeg + k) * ldb + gn;
    lb[u] = r * BKP + k;
    kb[u] = k;
  }
  double2 ra[NA], rb[NB];
  // slice at k0 into registers; FULL: all its BK k are inside the chunk
  auto gload = [&](int k0, auto full) {
    constexpr bool FULL = decltype(full)::value;
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      ra[u] = FULL || k0 + ka[u] < kend ? *pa[u] : make_double2(0.0, 0.0);
      pa[u] += BK;
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      rb[u] = FULL || k0 + kb[u] < kend ? *pb[u] : make_double2(0.0, 0.0);
      pb[u] += BMODE == 0 ? (long)BK : (long)BK * ldb;
    }
  };
  auto load = [&](int k0) {
    if (k0 + BK <= kend)
      gload(k0, std::true_type{});
    else if (k0 < kend)
      gload(k0, std::false_type{});
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int u = 0; u < NA; ++u) As[buf][la[u]] = ra[u];
#pragma unroll
    for (int u = 0; u < NB; ++u) Bs[buf][lb[u]] = rb[u];
  };
  const int lr = lane % 16;   // row (A) / column (B) inside a block
  const int lk = lane / 16;   // k inside a step of 4
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      double2 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = As[buf][(wm0 + i * 16 + lr) * BKP + kk + lk];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = Bs[buf][(wn0 + j * 16 + lr) * BKP + kk + lk];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          mfma(a[i].x, b[j].x, p[0][i][j]);
          if constexpr (RM == 1 || RM == 3) mfma(CJ ? a[i].y : -a[i].y, b[j].y, p[0][i][j]);
          if constexpr (RM == 3) {
            mfma(a[i].y, b[j].x, p[1][i][j]);
            mfma(CJ ? -a[i].x : a[i].x, b[j].y, p[1][i][j]);
          }
          if constexpr (RM == 2) mfma(a[i].x, b[j].y, p[1][i][j]);
          if constexpr (RM == 0) {
            mfma(a[i].y, b[j].y, p[1][i][j]);
            mfma(a[i].x + a[i].y, CJ ? b[j].x - b[j].y : b[j].x + b[j].y, p[2][i][j]);
          }
        }
    }
  };
  // one slice in flight: loaded during the MFMAs of the previous one
  load(kbeg);
  sstore(0);
  __syncthreads();
  int buf = 0, k0 = kbeg;
  for (; k0 + 2 * BK <= kend; k0 += BK) {
    gload(k0 + BK, std::true_type{});
    compute(buf);
    sstore(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  for (; k0 < kend; k0 += BK) {
    const bool more = k0 + BK < kend;
    if (more) load(k0 + BK);
    compute(buf);
    if (more) sstore(buf ^ 1);
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
          double2 *q = Cz + (long)gm * ldc + gn;
          double cr = p[0][i][j][r], ci = 0.0;
          if constexpr (RM >= 2) ci = p[1][i][j][r];
          if constexpr (RM == 0) {
            const double p1 = p[0][i][j][r], p2 = CJ ? -p[1][i][j][r] : p[1][i][j][r];
            cr = p1 - p2;
            ci = p[2][i][j][r] - p1 - p2;
          }
          if (accumulate) {
            const double2 v = *q;
            cr += v.x;
            ci += v.y;
          }
          *q = make_double2(cr, ci);
        }
      }
}

template <int BMODE, int RM, int BM, int BN, int BK, int WGM, int WGN>
hipError_t run_tile(const GemmDesc &g, hipStream_t s) {
  const int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
  const long total = (long)tm * tn * g.nsplit;
  if (total > (1L << 30)) return hipErrorInvalidValue;
  const int per_xcd = (int)((total + 7) / 8);
  const int kchunk = g.nsplit > 1 ? g.kchunk : g.K;
  hipLaunchKernelGGL((cgemm_kernel<BMODE, BM, BN, BK, RM, WGM, WGN, BMODE == 0>), dim3(8 * per_xcd),
                     dim3(64 * WGM * WGN), 0, s, reinterpret_cast<const double2 *>(g.A), g.lda,
                     reinterpret_cast<const double2 *>(g.B), g.ldb,
                     reinterpret_cast<double2 *>(g.C), g.ldc, g.M, g.N, g.K,
                     g.accumulate, kchunk, g.split_stride, tm, tn, (int)total, per_xcd);
  return hipGetLastError();
}

// 64 x 64 tiles with K slices of 8, or 16 x 64 with slices of 16 (cgemm_flat).
// Both add an element's terms in the order of k, so where the form (the number of
// real products) is given, the tile changes no bit of the result.  Four products
// exist on flat tiles only.
template <int BMODE, int RM> hipError_t run(const GemmDesc &g, hipStream_t s) {
  const bool flat = cgemm_flat(g.M, g.N, g.K, g.bmode);
  if constexpr (RM == 0) {
    if (g.form == 4 || (g.form == 0 && flat))
      return run_tile<BMODE, 3, 16, 64, 16, 1, 4>(g, s);
  }
  if (flat) return run_tile<BMODE, RM, 16, 64, 16, 1, 4>(g, s);
  return run_tile<BMODE, RM, 64, 64, 8, 2, 2>(g, s);
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

// Flat 16 x 64 tiles where the product is too small for 64 x 64 tiles to hide
// the latency of their slices behind each other's MFMAs, or where rows beyond M
// cost more than the flat tile's lower rate (about 1.35 times the time per
// padded element).  Measured, 64 x 64 -> 16 x 64 (us): 16 bands x 8 projectors,
// K 1 503, 6.8 -> 4.0; 64 x 128, K 1 791, 8.1 -> 6.2; 77 x 384, K 9 121,
// 57 -> 44; 256 x 512, K 7 127, 112 -> 127; without a split 128 x 128, K 128,
// 20.5 -> 9.2; 64 x 1 791, K 128, 21 -> 9.7; 77 x 9 121, K 384 (286 tiles of
// 64 x 64), 93 -> 50; 256 x 7 127, K 512 (448 tiles), 124 -> 151.
bool cgemm_flat(int M, int N, int K, int bmode) {
  const long t64 = (long)((M + 63) / 64) * ((N + 63) / 64);
  if (bmode == 0 ? (double)M * N * K < 5e8 : t64 < 384) return true;
  return 64 * ((M + 63) / 64) > 1.35 * 16 * ((M + 15) / 16);
}

int cgemm_form(int M, int N, int K, int bmode) { return cgemm_flat(M, N, K, bmode) ? 4 : 3; }

// The Gamma-point forms: RM = 1 for beta^H psi (bmode 0), RM = 2 for beta ps
// (bmode 1, A = ps real in complex storage).
hipError_t launch_cgemm(const GemmDesc &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipSuccess;
  if (g.ta != T_D2 || g.tb != T_D2 || g.tc != T_D2 || g.conjA || g.conjB != (g.bmode == 0))
    return hipErrorInvalidValue;
  if (g.rmode == 0) return g.bmode == 0 ? run<0, 0>(g, s) : run<1, 0>(g, s);
  if (g.rmode == 1 && g.bmode == 0) return run<0, 1>(g, s);
  if (g.rmode == 2 && g.bmode == 1) return run<1, 2>(g, s);
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
