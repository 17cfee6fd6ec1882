// Eigenpairs of the real symmetric tridiagonal matrix that the subspace solver's
// Householder reduction leaves: Sturm counts and multisection for the
// eigenvalues, twisted factorizations and inverse iteration for the vectors.
#include "eigh_common.h"

namespace qeh {
namespace {

// ---------------------------------------------------------------- tridiagonal eigenpairs
// Number of eigenvalues below x of rows [s, t) of T, scaled to 1/2 <= ||T|| < 1:
// of one block of the split T, or of all of T with its blocks joined by
// kSplitE ||T||.
// Sign changes of the principal minors p_i of T - x I, by the recurrence
// p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}: one fused multiply-add a row on
// the dependent chain, where the quotients p_i / p_{i-1} take a reciprocal
// estimate and two Newton steps.  T being scaled, a chunk of kSU rows grows the
// pair by at most 4^kSU, and, no e^2 being below (kSplitE / 2)^2, never takes both
// to zero; after each chunk the pair is scaled by a power of two.  (Over an e^2
// of zero it could: with d_i = x every later p would be a zero of either sign.)
// A zero p_i counts as positive: with p_{i+1} of the sign
// opposite to p_{i-1} the pair of rows has one change either way.  The
// operands (LDS) are read a chunk ahead.
constexpr int kSU = 8;
constexpr double kSplitE = 0.125 * kEps;
__device__ __forceinline__ int sturm_count(const double *d, const double *e2, int s, int t,
                                           double x) {
  double p1 = d[s] - x, p2 = 1.0;
  int c = __double2hiint(p1) < 0 ? 1 : 0;
  int i = s + 1;
  double dn[kSU], en[kSU];
  if (i + kSU <= t) {
#pragma unroll
    for (int u = 0; u < kSU; ++u) {
      dn[u] = d[i + u];
      en[u] = e2[i - 1 + u];
    }
  }
  for (; i + kSU <= t; i += kSU) {
    double dc[kSU], ec[kSU];
#pragma unroll
    for (int u = 0; u < kSU; ++u) {
      dc[u] = dn[u] - x;
      ec[u] = en[u];
    }
    if (i + 2 * kSU <= t) {
#pragma unroll
      for (int u = 0; u < kSU; ++u) {
        dn[u] = d[i + kSU + u];
        en[u] = e2[i + kSU - 1 + u];
      }
    }
#pragma unroll
    for (int u = 0; u < kSU; ++u) {
      const double p = fma(dc[u], p1, -(ec[u] * p2));
      c += (unsigned)(__double2hiint(p) ^ __double2hiint(p1)) >> 31;
      p2 = p1;
      p1 = p;
    }
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p1), fabs(p2)));
    p1 = __builtin_amdgcn_ldexp(p1, ex);
    p2 = __builtin_amdgcn_ldexp(p2, ex);
  }
  for (; i < t; ++i) {
    const double p = fma(d[i] - x, p1, -(e2[i - 1] * p2));
    c += (unsigned)(__double2hiint(p) ^ __double2hiint(p1)) >> 31;
    p2 = p1;
    p1 = p;
  }
  return c;
}

__device__ __forceinline__ double guard(double q, double pivmin) {
  return fabs(q) < pivmin ? -pivmin : q;
}

// deterministic start vector entry in [-1, 1) for row i of group member r
__device__ __forceinline__ double start_entry(int i, int r) {
  unsigned long long z = (unsigned long long)(i + 1) * 0x9E3779B97F4A7C15ull ^
                         (unsigned long long)(r + 1) * 0xC2B2AE3D27D4EB4Full;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// Solve (T_b - sigma I) x = x in place with the pivoted LU (dl, dd, du, du2,
// piv) of length m; tiny pivots replaced by +-tiny.
__device__ void lu_solve(const double *dl, const double *dd, const double *du, const double *du2,
                         const double *piv, int m, double tiny, double *x) {
  for (int i = 0; i + 1 < m; ++i) {
    if (piv[i] != 0.0) {
      const double a = x[i], b = x[i + 1];
      x[i] = b;
      x[i + 1] = a - dl[i] * b;
    } else {
      x[i + 1] -= dl[i] * x[i];
    }
  }
  auto piv_d = [&](int i) {
    const double v = dd[i];
    return fabs(v) < tiny ? copysign(tiny, v) : v;
  };
  x[m - 1] /= piv_d(m - 1);
  if (m > 1) x[m - 2] = (x[m - 2] - du[m - 2] * x[m - 1]) / piv_d(m - 2);
  for (int i = m - 3; i >= 0; --i) x[i] = (x[i] - du[i] * x[i + 1] - du2[i] * x[i + 2]) / piv_d(i);
}

// Gram-Schmidt of the columns of one group (tasks g0 .. g0+cnt-1 in block
// order, Z columns zc[task]) by one wave: each column against the earlier
// ones, then normalised.
__device__ void wave_mgs(double *Z, int ldz, const int *zc, int g0, int cnt, int s, int t) {
  const int lane = threadIdx.x & 63;
  for (int r = 0; r < cnt; ++r) {
    double *zr = Z + (long)zc[g0 + r] * ldz;
    for (int rr = 0; rr < r; ++rr) {
      const double *zq = Z + (long)zc[g0 + rr] * ldz;
      double dp = 0.0;
      for (int i = s + lane; i < t; i += 64) dp += zq[i] * zr[i];
      dp = wave_sum(dp);
      for (int i = s + lane; i < t; i += 64) zr[i] -= dp * zq[i];
    }
    double nn = 0.0;
    for (int i = s + lane; i < t; i += 64) nn += zr[i] * zr[i];
    nn = wave_sum(nn);
    const double inv = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
    for (int i = s + lane; i < t; i += 64) zr[i] *= inv;
  }
}

// The nb lowest eigenpairs of T (tri = d | e).  w[j] ascending, Z(:, j)
// (column-major, ldz >= n, real) orthonormal eigenvectors.  scr:
// eig_scratch_doubles(n) doubles.  info: 0, 1 (T not finite), 2 (fewer than
// nb eigenvalues found).  Two launches: PH = 0 over many workgroups finds the
// cut and the eigenvalues (each workgroup sets up T and the tasks itself, the
// same arithmetic in each, and bisects its share of the tasks), leaving the
// cut and the task eigenvalues in scr; PH = 1 takes them, sorts and groups them
// (again each workgroup by itself) and forms the eigenvectors of its share,
// TPW tasks or so.
// KM: largest order this instance takes (array sizes); NT threads.
template <int PH, int KM, int NT, int TPW>
__global__ __launch_bounds__(NT) void trieig_kernel(const double *tri, int n, int nb, double *w,
                                                     double *Z, int ldz, double *scr, int *info,
                                                     const int *info_chol) {
  if (*info_chol != 0) return;
  if (PH == 1 && *info != 0) return;
  if (PH == 0 && blockIdx.x == 0 && threadIdx.x == 0) *info = 0;
  double *tlam_g = scr + 7L * n * n;   // task eigenvalues, then the cut
  double *xcut_g = tlam_g + KM;
  __shared__ double sd[KM], se[KM], se2[KM];
  __shared__ int bst[KM + 1];    // block starts
  __shared__ int bof[KM + 1];    // first task of each block
  __shared__ double tlam[KM];    // task eigenvalue
  __shared__ int tblk[KM], tpos[KM];   // task block, sorted position
  __shared__ int gdeg[KM], gclo[KM];   // first task of the task's degenerate / close group
  constexpr int NW = NT / 64;
  constexpr int kSK = KM > NT ? KM : NT;   // sort keys (tasks <= KM, a power of two)
  __shared__ double key[kSK];
  __shared__ int kid[kSK];
  __shared__ double red[NW];
  __shared__ int sh_i[4];            // nblk, ntask, first qualifying multisection point / share
  __shared__ double sh_d[2];         // multisection bracket
  const int tid = threadIdx.x;
  const int wid = tid >> 6, lane = tid & 63;
  for (int i = tid; i < n; i += NT) {
    sd[i] = tri[i];
    se[i] = i + 1 < n ? tri[n + i] : 0.0;
  }
  __syncthreads();
  double md = 0.0, me = 0.0;
  for (int i = tid; i < n; i += NT) {
    md = fmax(md, fabs(sd[i]));
    me = fmax(me, fabs(se[i]));
  }
  md = block_max<NW>(md, red);
  me = block_max<NW>(me, red);
  double tnorm = md + 2.0 * me;
  if (!isfinite(tnorm) || nb < 1 || nb > n) {
    if (PH == 0 && blockIdx.x == 0 && tid == 0) *info = 1;
    return;
  }
  // T scaled by a power of two to 1/2 <= ||T|| < 1 (exact; the eigenvalues are
  // scaled back where they are written): the squares neither overflow nor lose
  // their digits
  const int tex = __builtin_amdgcn_frexp_exp(tnorm);
  tnorm = tnorm > 0.0 ? __builtin_amdgcn_ldexp(tnorm, -tex) : 1.0;
  // split where |e| is negligible; the squares there, which only the counts over
  // all of T read, move its eigenvalues by less than kEps ||T||
  double e2max = 0.0;
  for (int i = tid; i < n; i += NT) {
    sd[i] = __builtin_amdgcn_ldexp(sd[i], -tex);
    const double e = __builtin_amdgcn_ldexp(se[i], -tex);
    const bool split = fabs(e) <= kEps * tnorm;
    se[i] = split ? 0.0 : e;
    se2[i] = split ? kSplitE * tnorm * (kSplitE * tnorm) : e * e;
    e2max = fmax(e2max, se[i] * se[i]);
  }
  e2max = block_max<NW>(e2max, red);
  const double pivmin = kTiny * fmax(1.0, e2max);
  double lo = 1e300, hi = -1e300;
  for (int i = tid; i < n; i += NT) {
    const double r = fabs(se[i]) + (i > 0 ? fabs(se[i - 1]) : 0.0);
    lo = fmin(lo, sd[i] - r);
    hi = fmax(hi, sd[i] + r);
  }
  const double gl = block_min<NW>(lo, red) - 2.0 * kEps * tnorm - pivmin;
  const double gu = block_max<NW>(hi, red) + 2.0 * kEps * tnorm + pivmin;
  {
    // block starts in order: positions by ballots, waves and rounds added up
    int nbk = 1;
    if (tid == 0) bst[0] = 0;
    for (int i0 = 0; i0 + 1 < n; i0 += NT) {
      const int i = i0 + tid;
      const bool f = i + 1 < n && se[i] == 0.0;
      const unsigned long long m = __ballot(f);
      if (lane == 0) kid[wid] = __popcll(m);
      __syncthreads();
      int at = nbk;
      for (int v = 0; v < NW; ++v) {
        if (v < wid) at += kid[v];
        nbk += kid[v];
      }
      if (f) bst[at + __popcll(m & ((1ull << lane) - 1))] = i + 1;
      __syncthreads();
    }
    if (tid == 0) {
      bst[nbk] = n;
      sh_i[0] = nbk;
    }
  }
  __syncthreads();
  const int nblk = sh_i[0];
  // bracket the nb-th eigenvalue: count(lo) <= nb - 1 < count(hi)
  if (tid == 0) {
    sh_d[0] = gl;
    sh_d[1] = gu;
  }
  __syncthreads();
  if (PH == 0) {
    // (stops once exactly nb eigenvalues lie below the upper end: the cut then
    // selects the nb wanted ones and nothing else)
    int cup = n;   // count at the upper end
    for (int round = 0; round < 8; ++round) {
      const double a = sh_d[0], b = sh_d[1];
      if (b - a <= 2.0 * kEps * tnorm || cup == nb) break;   // uniform
      const double x = a + (b - a) * (double)(tid + 1) / (double)(NT + 1);
      const int c = sturm_count(sd, se2, 0, n, x);
      if (tid == 0) sh_i[2] = NT;
      __syncthreads();
      if (c > nb - 1) atomicMin(&sh_i[2], tid);   // first point above: order-free minimum
      __syncthreads();
      const int f = sh_i[2];
      if (tid == f) sh_i[3] = c;
      __syncthreads();
      if (f < NT) cup = sh_i[3];
      if (tid == 0) {
        const double xf = f < NT ? a + (b - a) * (double)(f + 1) / (double)(NT + 1) : b;
        const double xl = f > 0 ? a + (b - a) * (double)f / (double)(NT + 1) : a;
        sh_d[0] = xl;
        sh_d[1] = xf;
      }
      __syncthreads();
    }
  }
  const double xcut = PH == 0 ? sh_d[1] + 4.0 * kEps * tnorm + pivmin : *xcut_g;
  if (PH == 0 && blockIdx.x == 0 && tid == 0) *xcut_g = xcut;
  // eigenvalues of each block below the cut -> tasks
  for (int b = tid; b < nblk; b += NT) bof[b] = sturm_count(sd, se2, bst[b], bst[b + 1], xcut);
  __syncthreads();
  if (tid == 0) {
    int acc = 0;
    for (int b = 0; b < nblk; ++b) {
      const int c = bof[b];
      bof[b] = acc;
      acc += c;
    }
    bof[nblk] = acc;
    sh_i[1] = acc;
  }
  __syncthreads();
  const int ntask = sh_i[1];
  if (ntask < nb || ntask > KM) {
    if (PH == 0 && blockIdx.x == 0 && tid == 0) *info = 2;
    return;
  }
  for (int t = tid; t < ntask; t += NT) {   // last block whose first task is <= t
    int lb = 0, hb = nblk - 1;
    while (lb < hb) {
      const int md2 = (lb + hb + 1) >> 1;
      if (bof[md2] <= t) lb = md2;
      else hb = md2 - 1;
    }
    tblk[t] = lb;
  }
  __syncthreads();
  if (PH == 0) {
    // Start brackets.  When T is one block (the usual case) a task's local
    // index is its global one, and one pass of NT Sturm counts over
    // [gl, xcut] gives every task a bracket 1/(NT + 1) of that range wide
    // (count at the lower end <= index < count at the upper end).
    if (nblk == 1) {
      kid[tid] = sturm_count(sd, se2, 0, n,
                             gl + (xcut - gl) * (double)(tid + 1) / (double)(NT + 1));
      __syncthreads();
    }
    // Multisection, G lanes per task over all workgroups (the lanes of a
    // group adjacent in one wave; G a power of two <= 64): each round the
    // group's G points split the bracket into G + 1 parts and the first
    // point whose count exceeds the task's index becomes the upper end.
    // Every lane takes part in every round (one wave-wide ballot carries
    // the groups' comparisons), finished groups unchanged.
    const int gthreads = gridDim.x * NT;
    int G = 64;
    while (G > 1 && G * ntask > gthreads) G >>= 1;
    const int gt = blockIdx.x * NT + tid;
    // (more tasks than lanes, one lane each: rounds of gthreads tasks)
    for (int tb = 0; tb < ntask; tb += gthreads / G) {
    const int task = tb + gt / G, sub = gt % G;
    const bool real_task = task < ntask;
    const int b = real_task ? tblk[task] : 0;
    const int s = bst[b], t = bst[b + 1], loc = real_task ? task - bof[b] : 0;
    double a = gl, c = xcut;
    if (nblk == 1 && real_task) {
      int lo = 0, hi = NT;   // first point with count > loc (NT: none)
      while (lo < hi) {
        const int md = (lo + hi) >> 1;
        if (kid[md] > loc) hi = md;
        else lo = md + 1;
      }
      if (lo < NT) c = gl + (xcut - gl) * (double)(lo + 1) / (double)(NT + 1);
      if (lo > 0) a = gl + (xcut - gl) * (double)lo / (double)(NT + 1);
    }
    if (t - s == 1) a = c = sd[s];
    const int base = lane - sub;   // the group's first lane
    for (int it = 0; it < 160; ++it) {
      // (to eps ||T|| / 2, or no number left between; outer points may already
      // coincide with the ends)
      const double mid = 0.5 * (a + c);
      const bool act = real_task && c - a > 0.5 * kEps * tnorm && mid > a && mid < c;
      if (!__any(act)) break;
      const double x = a + (c - a) * (double)(sub + 1) / (double)(G + 1);
      const unsigned long long above =
          __ballot(sturm_count(sd, se2, s, t, x) > loc);
      // first point of the group above the index (G: none)
      const unsigned long long mine = (above >> base) & (G == 64 ? ~0ull : ((1ull << G) - 1));
      const int first = mine ? __builtin_ctzll(mine) : G;
      if (act) {
        const double na = first > 0 ? a + (c - a) * (double)first / (double)(G + 1) : a;
        const double nc = first < G ? a + (c - a) * (double)(first + 1) / (double)(G + 1) : c;
        a = na;
        c = nc;
      }
    }
    if (real_task && sub == 0) tlam_g[task] = 0.5 * (a + c);
    }
    return;
  }
  for (int i = tid; i < ntask; i += NT) tlam[i] = tlam_g[i];
  __syncthreads();
  // sort (value, task) pairs by value, task index breaking ties (bitonic over
  // KS keys, a power of two >= ntask)
  int KS = 2;
  while (KS < ntask) KS <<= 1;
  for (int e = tid; e < KS; e += NT) {
    key[e] = e < ntask ? tlam[e] : INFINITY;
    kid[e] = e;
  }
  for (int e = tid; e < KM; e += NT) tpos[e] = nb;   // not selected unless sorted below nb
  __syncthreads();
  for (int size = 2; size <= KS; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int e = tid; e < KS; e += NT) {
        const int p = e ^ stride;
        if (p > e) {
          const bool up = (e & size) == 0;
          const double ka = key[e], kb = key[p];
          const int ia = kid[e], ib = kid[p];
          const bool gt = ka > kb || (ka == kb && ia > ib);
          if (gt == up) {
            key[e] = kb;
            key[p] = ka;
            kid[e] = ib;
            kid[p] = ia;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int e = tid; e < ntask; e += NT)
    if (kid[e] < ntask) tpos[kid[e]] = e;
  __syncthreads();
  // groups within a block among the selected tasks (tasks of one block are
  // consecutive and ascending)
  for (int task = tid; task < ntask; task += NT)
    if (tpos[task] < nb) {
      int g = task;
      while (g > bof[tblk[task]] && tpos[g - 1] < nb && tlam[g] - tlam[g - 1] <= kDegRel * tnorm)
        --g;
      gdeg[task] = g;
      g = task;
      while (g > bof[tblk[task]] && tpos[g - 1] < nb && tlam[g] - tlam[g - 1] <= kCloseRel * tnorm)
        --g;
      gclo[task] = g;
    }
  __syncthreads();
  // The workgroup's share: the tasks whose close group begins in its range of
  // TPW tasks (groups stay whole; a range of consecutive tasks).
  if (tid == 0) {
    sh_i[2] = ntask;
    sh_i[3] = 0;
  }
  __syncthreads();
  for (int task = tid; task < ntask; task += NT)
    if (tpos[task] < nb && gclo[task] / TPW == (int)blockIdx.x) {
      atomicMin(&sh_i[2], task);
      atomicMax(&sh_i[3], task + 1);
    }
  __syncthreads();
  const int tb = sh_i[2], te = sh_i[3];
  const long ls = n;   // per-task scratch stride
  const long kTS = ls;                  // row stride of the pivot arrays (tasks <= n)
  double *twp = scr;                    // [n][task] D+ (top-down pivots)
  double *twm = scr + ls * ls;          // [n][task] D- (bottom-up pivots)
  double *lu = scr + 2 * ls * ls;       // [task][5 n] pivoted LU (group leaders)
  const double dtiny = kEps * tnorm;
  auto in_group = [&](int t) {   // selected task t is in a degenerate group of >= 2
    return gdeg[t] != t || (t + 1 < bof[tblk[t] + 1] && tpos[t + 1] < nb && gdeg[t + 1] == t);
  };
  if constexpr (KM <= 128) {
    // pass 1 with the pivots in LDS, TPW tasks at a time: the top-down and the
    // bottom-up recurrences in two waves, one lane a task; everything else 16
    // lanes a task
    constexpr int P = KM + 1, kL = NT / TPW;
    static_assert(kL == 16, "a task's lanes are a row of 16");
    __shared__ double pv[2][TPW][P];
    __shared__ int pr[TPW];
    __shared__ double pn[2][TPW];
    for (int t0 = tb; t0 < te; t0 += TPW) {
      __syncthreads();
      const int side = wid;   // 0: from the top, 1: from the bottom
      const int mine = t0 + lane;
      if (side < 2 && lane < TPW && mine < te && tpos[mine] < nb && !in_group(mine)) {
        const int s = bst[tblk[mine]], t = bst[tblk[mine] + 1], m = t - s;
        const double lam = tlam[mine];
        double *q = pv[side][lane];
        if (side == 0) {
          double qp = sd[s] - lam;
          q[0] = qp;
          for (int i = 1; i < m; ++i) {
            qp = sd[s + i] - lam - quot(se2[s + i - 1], guard(qp, pivmin));
            q[i] = qp;
          }
        } else {
          double qm = sd[t - 1] - lam;
          q[m - 1] = qm;
          for (int i = m - 2; i >= 0; --i) {
            qm = sd[s + i] - lam - quot(se2[s + i], guard(qm, pivmin));
            q[i] = qm;
          }
        }
      }
      __syncthreads();
      const int slot = tid / kL, l = tid % kL, task = t0 + slot;
      const bool single = task < te && tpos[task] < nb && !in_group(task);
      int s = 0, m = 0;
      if (single) {
        s = bst[tblk[task]];
        m = bst[tblk[task] + 1] - s;
      }
      // the twist: the first row of least |gamma|
      double best = INFINITY;
      int r = 0;
      for (int i = l; i < m; i += kL) {
        const double gm = fabs(pv[0][slot][i] + pv[1][slot][i] - (sd[s + i] - tlam[task]));
        if (gm < best) {
          best = gm;
          r = i;
        }
      }
      for (int o = kL / 2; o > 0; o >>= 1) {
        const double ob = __shfl_xor(best, o);
        const int orow = __shfl_xor(r, o);
        if (ob < best || (ob == best && orow < r)) {
          best = ob;
          r = orow;
        }
      }
      if (l == 0) pr[slot] = r;
      __syncthreads();
      // the unnormalised vector (entry r = 1) replaces the pivots it is formed from
      if (side < 2 && lane < TPW && mine < te && tpos[mine] < nb && !in_group(mine)) {
        const int s1 = bst[tblk[mine]], m1 = bst[tblk[mine] + 1] - s1, r1 = pr[lane];
        double *q = pv[side][lane];
        double zc = 1.0, nn = 0.0;
        if (side == 0) {
#pragma unroll 4
          for (int i = r1 - 1; i >= 0; --i) {
            zc = -quot(se[s1 + i], guard(q[i], pivmin)) * zc;
            q[i] = zc;
            nn += zc * zc;
          }
        } else {
#pragma unroll 4
          for (int i = r1; i + 1 < m1; ++i) {
            zc = -quot(se[s1 + i], guard(q[i + 1], pivmin)) * zc;
            q[i + 1] = zc;
            nn += zc * zc;
          }
        }
        pn[side][lane] = nn;
      }
      __syncthreads();
      if (single) {
        double *z = Z + (long)tpos[task] * ldz;
        const double inv = 1.0 / sqrt(1.0 + pn[0][slot] + pn[1][slot]);
        for (int i = l; i < n; i += kL) {
          const int li = i - s;
          const double v = li < 0 || li >= m ? 0.0
                           : li < r          ? pv[0][slot][li]
                           : li == r         ? 1.0
                                             : pv[1][slot][li];
          z[i] = v * inv;
        }
      }
    }
  }
  // pass 1: twisted vectors (singletons); LU of the degenerate groups (leaders)
  for (int task = tb + tid; task < te; task += NT) {
    if (tpos[task] >= nb) continue;
    const int b = tblk[task], s = bst[b], t = bst[b + 1], m = t - s;
    double *z = Z + (long)tpos[task] * ldz;
    const double lam = tlam[task];
    if (in_group(task))
      for (int i = 0; i < n; ++i)
        if (i < s || i >= t) z[i] = 0.0;
    if (!in_group(task)) {
      if (KM <= 128) {   // (done above)
      } else if (m == 1) {
        for (int i = 0; i < n; ++i) z[i] = i == s ? 1.0 : 0.0;
      } else {
        // pivots stored row-major over the tasks ([i][task]): the lanes of a
        // wave touch consecutive addresses at each step
        // (the top-down and bottom-up recurrences interleaved: two
        // independent chains)
        double *dp = twp + task, *dm = twm + task;
        double qp = sd[s] - lam, qm = sd[t - 1] - lam;
        dp[0] = qp;
        dm[(m - 1) * kTS] = qm;
        for (int i = 1; i < m; ++i) {
          const int j = m - 1 - i;
          qp = sd[s + i] - lam - quot(se2[s + i - 1], guard(qp, pivmin));
          qm = sd[s + j] - lam - quot(se2[s + j], guard(qm, pivmin));
          dp[i * kTS] = qp;
          dm[j * kTS] = qm;
        }
        int r = 0;
        double best = INFINITY;
#pragma unroll 8
        for (int i = 0; i < m; ++i) {
          const double gm = fabs(dp[i * kTS] + dm[i * kTS] - (sd[s + i] - lam));
          if (gm < best) {
            best = gm;
            r = i;
          }
        }
        // the unnormalised vector (entry r = 1) replaces the pivots it is
        // formed from (coalesced), and goes to Z once, normalised, with the
        // zeros outside the block (one strided pass)
        double zc = 1.0, nn = 1.0;
#pragma unroll 8
        for (int i = r - 1; i >= 0; --i) {
          zc = -quot(se[s + i], guard(dp[i * kTS], pivmin)) * zc;
          dp[i * kTS] = zc;
          nn += zc * zc;
        }
        zc = 1.0;
#pragma unroll 8
        for (int i = r; i + 1 < m; ++i) {
          zc = -quot(se[s + i], guard(dm[(i + 1) * kTS], pivmin)) * zc;
          dm[(i + 1) * kTS] = zc;
          nn += zc * zc;
        }
        const double inv = 1.0 / sqrt(nn);
#pragma unroll 8
        for (int i = 0; i < n; ++i) {
          const int li = i - s;
          const double v = li < 0 || li >= m ? 0.0 : li < r ? dp[li * kTS] : li == r ? 1.0 : dm[li * kTS];
          z[i] = v * inv;
        }
      }
    } else if (gdeg[task] == task) {
      // pivoted LU of T_b - lam I (LAPACK gttrf order)
      double *dl = lu + (long)task * 5 * ls, *dd = dl + ls, *du = dd + ls, *du2 = du + ls,
             *pv = du2 + ls;
      for (int i = 0; i < m; ++i) dd[i] = sd[s + i] - lam;
      for (int i = 0; i + 1 < m; ++i) {
        dl[i] = se[s + i];
        du[i] = se[s + i];
        pv[i] = 0.0;
      }
      for (int i = 0; i + 2 < m; ++i) du2[i] = 0.0;
      for (int i = 0; i + 1 < m; ++i) {
        if (fabs(dd[i]) >= fabs(dl[i])) {
          const double f = dd[i] != 0.0 ? dl[i] / dd[i] : 0.0;
          dl[i] = f;
          dd[i + 1] -= f * du[i];
        } else {
          const double f = dd[i] / dl[i];
          dd[i] = dl[i];
          dl[i] = f;
          const double tmp = du[i];
          du[i] = dd[i + 1];
          dd[i + 1] = tmp - f * dd[i + 1];
          if (i + 2 < m) {
            du2[i] = du[i + 1];
            du[i + 1] = -f * du[i + 1];
          }
          pv[i] = 1.0;
        }
      }
    }
  }
  __syncthreads();
  // passes 2-5: two sweeps of inverse iteration for the degenerate groups,
  // each followed by Gram-Schmidt within the group (one wave per group)
  for (int sweep = 0; sweep < 2; ++sweep) {
    for (int task = tb + tid; task < te; task += NT) {
      if (tpos[task] >= nb || !in_group(task)) continue;
      const int b = tblk[task], s = bst[b], t = bst[b + 1], m = t - s;
      const int ld0 = gdeg[task];
      const double *dl = lu + (long)ld0 * 5 * ls, *dd = dl + ls, *du = dd + ls, *du2 = du + ls,
                   *pv = du2 + ls;
      double *z = Z + (long)tpos[task] * ldz + s;
      if (sweep == 0)
        for (int i = 0; i < m; ++i) z[i] = start_entry(i, task - ld0);
      lu_solve(dl, dd, du, du2, pv, m, dtiny, z);
      double nn = 0.0;
      for (int i = 0; i < m; ++i) nn += z[i] * z[i];
      const double inv = nn > 0.0 && isfinite(nn) ? 1.0 / sqrt(nn) : 0.0;
      for (int i = 0; i < m; ++i) z[i] *= inv;
    }
    __syncthreads();
    // group leaders, dealt to waves in task order
    for (int t0 = tb + wid; t0 < te; t0 += NW) {
      if (tpos[t0] >= nb || gdeg[t0] != t0 || !in_group(t0)) continue;
      int cnt = 1;
      while (t0 + cnt < bof[tblk[t0] + 1] && tpos[t0 + cnt] < nb && gdeg[t0 + cnt] == t0) ++cnt;
      wave_mgs(Z, ldz, tpos, t0, cnt, bst[tblk[t0]], bst[tblk[t0] + 1]);
    }
    __syncthreads();
  }
  // close groups: Gram-Schmidt in block order (one wave per group)
  for (int t0 = tb + wid; t0 < te; t0 += NW) {
    if (tpos[t0] >= nb || gclo[t0] != t0) continue;
    int cnt = 1;
    while (t0 + cnt < bof[tblk[t0] + 1] && tpos[t0 + cnt] < nb && gclo[t0 + cnt] == t0) ++cnt;
    if (cnt > 1) wave_mgs(Z, ldz, tpos, t0, cnt, bst[tblk[t0]], bst[tblk[t0] + 1]);
  }
  if (blockIdx.x == 0)
    for (int task = tid; task < ntask; task += NT)
      if (tpos[task] < nb) w[tpos[task]] = __builtin_amdgcn_ldexp(tlam[task], tex);
}

}  // namespace

size_t eig_scratch_doubles(int n) { return (size_t)7 * n * n + kEMaxN + 8; }

hipError_t launch_trieig(const double *tri, int n, int nb, double *w, double *Z, int ldz,
                         double *scr, int *info, const int *info_chol, bool wide, hipStream_t s) {
  if (n < 1 || n > kEMaxN || nb < 1 || nb > n || ldz < n) return hipErrorInvalidValue;
  // Eigenvalues on 256-thread workgroups, 64 lanes per wanted one over up to 128
  // of them (wide): four Sturm recurrences a SIMD already share its issue, so
  // 1024 threads on a CU took four times as long per round, and one
  // workgroup of 256 (narrow) does less work in total than one of 1024, a
  // round gaining log2(G + 1) bits from G lanes.  Vectors 16 tasks a workgroup
  // (LDS holds their pivots) or, above order 128, 64 (a wave's coalesced
  // accesses).  64 of about 120: eigenvalues 162 -> 47 us, vectors 127 -> 40 us
  // (one workgroup of 1024 threads each, the vectors' pivots in global memory).
  // (Instances sized for the order: the 2 048-task arrays measured 20% slower
  // on orders <= 512.)
  const int g = wide ? max(1, min(128, (nb * 64 + 255) / 256)) : 1;
  auto go = [&](auto k0, auto k1, int tpw) {
    hipLaunchKernelGGL(k0, dim3(g), dim3(256), 0, s, tri, n, nb, w, Z, ldz, scr, info, info_chol);
    hipLaunchKernelGGL(k1, dim3((n + tpw - 1) / tpw), dim3(256), 0, s, tri, n, nb, w, Z, ldz, scr,
                       info, info_chol);
  };
  if (n <= 128) go(trieig_kernel<0, 128, 256, 16>, trieig_kernel<1, 128, 256, 16>, 16);
  else if (n <= 512) go(trieig_kernel<0, 512, 256, 64>, trieig_kernel<1, 512, 256, 64>, 64);
  else if (n <= 1024) go(trieig_kernel<0, 1024, 256, 64>, trieig_kernel<1, 1024, 256, 64>, 64);
  else go(trieig_kernel<0, kEMaxN, 256, 64>, trieig_kernel<1, kEMaxN, 256, 64>, 64);
  return hipGetLastError();
}

}  // namespace qeh
