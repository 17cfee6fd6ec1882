// Single-precision projector products (mixed form: becp = beta^H psi and
// hpsi += beta ps, the pseudopotential kernels of section "Evolution of the
// GPU-enabled version") on the bf16 matrix units, without giving up any
// single-precision input bit.
//
// Each FP32 operand value x is written as x = x0 + x1 + x2 with bf16 parts
// (round to nearest, remainders exact in FP32): 3 x 8 bits carry the 24-bit
// significand.  (Values above 3.396e38, the top 0.2% of the float range, round to
// an infinite first part.)  A product is the six part products whose size is at least
// 2^-17 of the whole, x0 y0 + x0 y1 + x1 y0 + x1 y1 + x0 y2 + x2 y0, each exact
// and accumulated in FP32 by the MFMA; the three left out are below 2^-24.
// The bf16 unit runs 16 times the FP32 one's rate, so six products leave it
// 2.7 times as fast, and a K step of 16 costs 6 roundings of the accumulator
// where the FP32 instruction (k = 2) takes 8.
//
// A complex product takes four real ones (re re, im im, re im, im re) into two
// accumulator sets; the three-product form would need the operand sums split
// and staged as well.  Gamma forms: RM = 1, only Re C is wanted (two products,
// one accumulator set); RM = 2, A is real (two products, two sets).
//
// One workgroup: WGM x WGN waves, each a (32 TM) x (32 TN) block of C from
// 32 x 32 x 16 MFMAs.  While the MFMAs of one K slice of 16 run from LDS, the
// next slice is split from registers into the other LDS buffer and the one
// after loaded: one barrier per slice, and the splitting (11 vector
// instructions per two values) shares the SIMD with the MFMAs.  LDS holds
// 16-byte units of eight k values, [part][re, im][k half][row], so fragment
// reads and the stores touch consecutive units (no bank conflicts).
//
// Bound: the bf16 matrix rate under load (1.22 PFLOP/s for a library product
// of 8192^3 random values here; the complex products reach 1.1 PFLOP/s of part
// products) and, at Gamma, which does half the MFMA work per staged value, the
// splitting.  Measured, FP32 MFMA kernel (16 x 16 x 4 or 32 x 32 x 2) -> this
// one, beta^H psi / beta ps:
//   202 bands x 404 projectors, 5 614 plane waves    58 -> 42 / 68 -> 43 us
//   128 x 512, 23 976                               109 -> 71 / 124 -> 83 us
//   64 x 2048, 74 047, Gamma                        443 -> 282 / 482 -> 351 us
//   128 x 6144, 93 225, Gamma                  2.77 -> 1.62 / 2.82 -> 1.70 ms
// (kernel traces of H psi on one card); against FP64 products of the same FP32
// inputs the relative error of beta^H psi fell from 5.0e-7 to 1.8e-7 (128 x 512) and
// from 1.2e-6 to 6.0e-7 (128 x 6144), of beta ps from 5.8e-7 to 4.9e-7 and 1.4e-6 to
// 1.2e-6.
#include <algorithm>
#include <type_traits>

#include "cplx.h"
#include "qeh_internal.h"

namespace qeh {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

constexpr int kBK = 16;     // k per slice (one MFMA step)

// four floats at an address aligned to 8 bytes (rows start at any complex element)
struct __attribute__((packed, aligned(8))) Float4 {
  float x, y, z, w;
};
struct __attribute__((packed, aligned(4))) Real4 {
  float x, y, z, w;
};

// the three bf16 parts of a and b, each pair packed
struct Parts {
  unsigned p0, p1, p2;
};
__device__ __forceinline__ Parts split2(float a, float b) {
  Parts r;
  r.p0 = __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{a, b}), bf16x2));
  const float a1 = a - __builtin_bit_cast(float, r.p0 << 16);   // remainders, exact
  const float b1 = b - __builtin_bit_cast(float, r.p0 & 0xffff0000u);
  r.p1 = __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{a1, b1}), bf16x2));
  const float a2 = a1 - __builtin_bit_cast(float, r.p1 << 16);
  const float b2 = b1 - __builtin_bit_cast(float, r.p1 & 0xffff0000u);
  r.p2 = __builtin_bit_cast(unsigned, __builtin_convertvector((floatx2{a2, b2}), bf16x2));
  return r;
}

__device__ __forceinline__ void mfma(uintx4 a, uintx4 b, floatx16 &c) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                              __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The six part products of two split fragments, small ones first.  The five
// small ones go to an accumulator set of their own (d): the large one then
// rounds c once per step instead of six times.
template <int TM, int TN>
__device__ __forceinline__ void mul6(const uintx4 (&a)[TM][3], const uintx4 (&b)[TN][3],
                                     floatx16 (&c)[TM][TN], floatx16 (&d)[TM][TN]) {
  constexpr int pa[5] = {2, 0, 1, 1, 0};
  constexpr int pb[5] = {0, 2, 1, 0, 1};
#pragma unroll
  for (int p = 0; p < 5; ++p)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) mfma(a[i][pa[p]], b[j][pb[p]], d[i][j]);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) mfma(a[i][0], b[j][0], c[i][j]);
}

// Four consecutive k of one K-contiguous row, the first n of them valid (all
// when FULL): real and imaginary parts.
template <bool FULL>
__device__ __forceinline__ void load4(const float2 *p, int n, float (&re)[4], float (&im)[4]) {
  if constexpr (FULL) {
    const Float4 u = *reinterpret_cast<const Float4 *>(p);
    const Float4 v = *reinterpret_cast<const Float4 *>(p + 2);
    re[0] = u.x, im[0] = u.y, re[1] = u.z, im[1] = u.w;
    re[2] = v.x, im[2] = v.y, re[3] = v.z, im[3] = v.w;
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float2 v = q < n ? p[q] : make_float2(0.f, 0.f);
      re[q] = v.x;
      im[q] = v.y;
    }
  }
}
template <bool FULL>
__device__ __forceinline__ void load4(const double2 *p, int n, float (&re)[4], float (&im)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double2 v = FULL || q < n ? p[q] : make_double2(0.0, 0.0);
    re[q] = (float)v.x;
    im[q] = (float)v.y;
  }
}
template <bool FULL>
__device__ __forceinline__ void load4(const float *p, int n, float (&re)[4], float (&im)[4]) {
  if constexpr (FULL) {
    const Real4 u = *reinterpret_cast<const Real4 *>(p);
    re[0] = u.x, re[1] = u.y, re[2] = u.z, re[3] = u.w;
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) re[q] = q < n ? p[q] : 0.f;
  }
}

template <typename T> struct is_real { static constexpr bool value = false; };
template <> struct is_real<float> { static constexpr bool value = true; };

// BMODE 0: B element (k, n) at B[n ldb + k], conjugated (beta^H psi);
// BMODE 1: at B[k ldb + n] (beta ps).
template <typename TA, typename TC, int BMODE, int RM, int TM, int TN, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN)
void split_gemm_kernel(
    const TA *__restrict__ A, long lda, const float2 *__restrict__ B, long ldb,
    TC *__restrict__ C, long ldc, int M, int N, int K, int accumulate, int kchunk,
    long split_stride, int tiles_m, int tiles_n, int ntiles, int per_xcd) {
  constexpr int kThreads = 64 * WGM * WGN;
  constexpr int BM = 32 * TM * WGM, BN = 32 * TN * WGN;
  constexpr bool AREAL = is_real<TA>::value;
  static_assert(AREAL == (RM == 2), "a real A is the RM = 2 form");
  constexpr int CA = AREAL ? 1 : 2;           // components of A in LDS
  constexpr int NCA = 4 * BM / kThreads, NCB = 4 * BN / kThreads;   // 4-k chunks per thread
  static_assert(NCA * kThreads == 4 * BM && NCB * kThreads == 4 * BN, "tile / thread mismatch");
  __shared__ uintx4 As[2][3][CA][2][BM];   // [buffer][part][re, im][k half][row]
  __shared__ uintx4 Bs[2][3][2][2][BN];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  // workgroup ids are dealt round-robin to the 8 XCDs (each with its own L2):
  // each XCD gets a contiguous run of (m tile fastest, n tile, K slice)
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
  TC *Cz = C + (long)kz * split_stride;

  // sums of the large and of the small part products (beta ps: its K, the
  // projectors, is short; one set takes both)
  floatx16 cr[TM][TN], ci[TM][TN], dr[TM][TN], di[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        cr[i][j][e] = 0.f;
        ci[i][j][e] = 0.f;
        dr[i][j][e] = 0.f;
        di[i][j][e] = 0.f;
      }

  // K-contiguous operands: chunk (row, kq) = four k of one row; four lanes
  // cover a row's 16 k (128 bytes), a wave 16 rows.  Rows beyond M / N repeat
  // the last one (their results are not stored), so whole slices load
  // without masks.
  constexpr int kRows = kThreads / 4;
  const int kq = tid & 3;
  const int crow = tid >> 2;
  const TA *pa[NCA];
#pragma unroll
  for (int u = 0; u < NCA; ++u)
    pa[u] = A + (long)min(m0 + crow + kRows * u, M - 1) * lda + (kbeg + 4 * kq);
  // BMODE 1 B: chunk (n, quarter) = four k of one column, lanes along n
  const float2 *pb[NCB];
#pragma unroll
  for (int u = 0; u < NCB; ++u) {
    if constexpr (BMODE == 0) {
      pb[u] = B + (long)min(n0 + crow + kRows * u, N - 1) * ldb + (kbeg + 4 * kq);
    } else {
      const int e = tid + u * kThreads;
      pb[u] = B + (long)(kbeg + 4 * (e / BN)) * ldb + min(n0 + e % BN, N - 1);
    }
  }
  struct Slice {
    float are[NCA][4], aim[NCA][4], bre[NCB][4], bim[NCB][4];
  };

  // slice at k0 into registers; FULL: all its 16 k are inside the chunk
  auto gload = [&](Slice &r, int k0, auto full) {
    constexpr bool FULL = decltype(full)::value;
    const int n = kend - (k0 + 4 * kq);
#pragma unroll
    for (int u = 0; u < NCA; ++u) {
      load4<FULL>(pa[u], n, r.are[u], r.aim[u]);
      pa[u] += kBK;
    }
#pragma unroll
    for (int u = 0; u < NCB; ++u) {
      if constexpr (BMODE == 0) {
        load4<FULL>(pb[u], n, r.bre[u], r.bim[u]);
        pb[u] += kBK;
      } else {
        const int nb = kend - (k0 + 4 * ((tid + u * kThreads) / BN));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float2 v = FULL || q < nb ? pb[u][(long)q * ldb] : make_float2(0.f, 0.f);
          r.bre[u][q] = v.x;
          r.bim[u][q] = v.y;
        }
        pb[u] += (long)kBK * ldb;
      }
    }
  };
  // four k of one component: 8 bytes per part at unit (k half, row)
  auto put4 = [&](uintx4 *base, long pstride, int off, const float (&v)[4]) {
    const Parts a = split2(v[0], v[1]), b = split2(v[2], v[3]);
    uintx2 *q = reinterpret_cast<uintx2 *>(base) + off;
    q[0] = uintx2{a.p0, b.p0};
    q[2 * pstride] = uintx2{a.p1, b.p1};
    q[4 * pstride] = uintx2{a.p2, b.p2};
  };
  auto sstore = [&](const Slice &r, int buf) {
#pragma unroll
    for (int u = 0; u < NCA; ++u) {
      const int off = 2 * ((kq >> 1) * BM + crow + kRows * u) + (kq & 1);
      put4(&As[buf][0][0][0][0], CA * 2 * BM, off, r.are[u]);
      if constexpr (!AREAL) put4(&As[buf][0][CA - 1][0][0], CA * 2 * BM, off, r.aim[u]);
    }
#pragma unroll
    for (int u = 0; u < NCB; ++u) {
      const int e = tid + u * kThreads;
      const int q = BMODE == 0 ? kq : e / BN;
      const int row = BMODE == 0 ? crow + kRows * u : e % BN;
      const int off = 2 * ((q >> 1) * BN + row) + (q & 1);
      put4(&Bs[buf][0][0][0][0], 4 * BN, off, r.bre[u]);
      put4(&Bs[buf][0][1][0][0], 4 * BN, off, r.bim[u]);
    }
  };

  const int kh = lane >> 5;
  const int arow = (wave / WGN) * 32 * TM + (lane & 31);
  const int brow = (wave % WGN) * 32 * TN + (lane & 31);
  auto lda_frag = [&](int buf, int c, uintx4 (&f)[TM][3]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int p = 0; p < 3; ++p) f[i][p] = As[buf][p][c][kh][arow + 32 * i];
  };
  auto ldb_frag = [&](int buf, int c, uintx4 (&f)[TN][3]) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int p = 0; p < 3; ++p) f[j][p] = Bs[buf][p][c][kh][brow + 32 * j];
  };
  auto compute = [&](int buf) {
    floatx16 (&sr)[TM][TN] = BMODE == 0 ? dr : cr;
    floatx16 (&si)[TM][TN] = BMODE == 0 ? di : ci;
    uintx4 ar[TM][3], ai[TM][3], bb[TN][3];
    lda_frag(buf, 0, ar);
    ldb_frag(buf, 0, bb);
    if constexpr (RM == 2) {   // A real
      mul6<TM, TN>(ar, bb, cr, sr);
      ldb_frag(buf, 1, bb);
      mul6<TM, TN>(ar, bb, ci, si);
    } else if constexpr (RM == 1) {   // Re(A conj B)
      mul6<TM, TN>(ar, bb, cr, sr);
      lda_frag(buf, 1, ai);
      ldb_frag(buf, 1, bb);
      mul6<TM, TN>(ai, bb, cr, sr);
    } else {
      lda_frag(buf, 1, ai);
      mul6<TM, TN>(ar, bb, cr, sr);
      mul6<TM, TN>(ai, bb, ci, si);
      ldb_frag(buf, 1, bb);
      // conj B (BMODE 0): cr += ai bi, ci -= ar bi; else cr -= ai bi, ci += ar bi
      uintx4 (&neg)[TM][3] = BMODE == 0 ? ar : ai;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p) neg[i][p] ^= 0x80008000u;
      mul6<TM, TN>(ai, bb, cr, sr);
      mul6<TM, TN>(ar, bb, ci, si);
    }
  };

  // One slice ahead in LDS, one in registers: while the MFMAs of slice t run,
  // slice t + 1 is split and stored and slice t + 2 loaded.
  const int nsl = (kend - kbeg + kBK - 1) / kBK;   // slices, the last one possibly short
  const int nfull = max(0, kend - kbeg) / kBK;     // whole slices
  Slice r;
  auto load = [&](int t) {
    if (t < nfull)
      gload(r, kbeg + t * kBK, std::true_type{});
    else if (t < nsl)
      gload(r, kbeg + t * kBK, std::false_type{});
  };
  load(0);
  if (nsl > 0) sstore(r, 0);
  load(1);
  __syncthreads();
  int t = 0;
  for (; t + 2 < nfull; ++t) {
    compute(t & 1);
    sstore(r, (t + 1) & 1);
    gload(r, 0, std::true_type{});
    __syncthreads();
  }
  for (; t < nsl; ++t) {
    compute(t & 1);
    if (t + 1 < nsl) sstore(r, (t + 1) & 1);
    load(t + 2);
    __syncthreads();
  }

  // 32 x 32 block: column lane % 32, entry e = row (e % 4) + 8 (e / 4) + 4 (lane / 32)
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int gm = m0 + (wave / WGN) * 32 * TM + 32 * i + (e % 4) + 8 * (e / 4) + 4 * kh;
        const int gn = n0 + brow + 32 * j;
        if (gm < M && gn < N) {
          using RC = typename real_of<TC>::type;
          TC *p = Cz + (long)gm * ldc + gn;
          TC v;
          v.x = static_cast<RC>(BMODE == 0 ? cr[i][j][e] + dr[i][j][e] : cr[i][j][e]);
          v.y = RM == 1 ? RC(0)
                : static_cast<RC>(BMODE == 0 ? ci[i][j][e] + di[i][j][e] : ci[i][j][e]);
          if (accumulate) {   // the add happens in the result's precision
            const TC o = *p;
            v.x = o.x + v.x;
            v.y = o.y + v.y;
          }
          *p = v;
        }
      }
}

template <typename TA, typename TC, int BMODE, int RM, int TM, int TN, int WGM, int WGN>
hipError_t run_split(const GemmDesc &g, hipStream_t s) {
  constexpr int BM = 32 * TM * WGM, BN = 32 * TN * WGN;
  const int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
  const long total = (long)tm * tn * g.nsplit;
  if (total > (1L << 30)) return hipErrorInvalidValue;
  const int per_xcd = (int)((total + 7) / 8);
  const int kchunk = g.nsplit > 1 ? g.kchunk : g.K;
  hipLaunchKernelGGL((split_gemm_kernel<TA, TC, BMODE, RM, TM, TN, WGM, WGN>),
                     dim3(8 * per_xcd), dim3(64 * WGM * WGN), 0, s,
                     reinterpret_cast<const TA *>(g.A), g.lda,
                     reinterpret_cast<const float2 *>(g.B), g.ldb, reinterpret_cast<TC *>(g.C),
                     g.ldc, g.M, g.N, g.K, g.accumulate, kchunk, g.split_stride, tm, tn,
                     (int)total, per_xcd);
  return hipGetLastError();
}

template <typename TA, typename TC, int BMODE, int RM>
hipError_t run_split_tile(const GemmDesc &g, hipStream_t s) {
  switch (g.tile) {
    case 0: return run_split<TA, TC, BMODE, RM, 1, 1, 2, 2>(g, s);   // 64 x 64
    case 1: return run_split<TA, TC, BMODE, RM, 1, 2, 2, 2>(g, s);   // 64 x 128
    case 2: return run_split<TA, TC, BMODE, RM, 2, 1, 2, 4>(g, s);   // 128 x 128, eight waves
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_split_gemm(const GemmDesc &g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipSuccess;
  if (g.tb != T_F2 || g.conjA) return hipErrorInvalidValue;
  if (g.bmode == 0 && g.conjB && g.tc == T_F2 && !g.accumulate) {   // beta^H psi
    if (g.rmode == 0)
      return g.ta == T_D2 ? run_split_tile<double2, float2, 0, 0>(g, s)
                          : run_split_tile<float2, float2, 0, 0>(g, s);
    if (g.rmode == 1)
      return g.ta == T_D2 ? run_split_tile<double2, float2, 0, 1>(g, s)
                          : run_split_tile<float2, float2, 0, 1>(g, s);
  }
  if (g.bmode == 1 && !g.conjB && g.tc == T_D2) {   // beta ps
    if (g.rmode == 0 && g.ta == T_F2) return run_split_tile<float2, double2, 1, 0>(g, s);
    if (g.rmode == 2 && g.ta == T_F1) return run_split_tile<float, double2, 1, 2>(g, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace qeh
