// Two-factor plane pass, single precision (see plane2.h), and its geometry.
#include "plane2.h"

namespace qeh {

hipError_t launch_k2_two_f32(const qeh_ctx *c, int nbk) {
  switch (c->n1) {
#define QEH_TWO_CASE(NN) \
  case NN: return plane2::launch<float2, NN>(c, nbk);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return hipErrorInvalidValue;
  }
}

namespace {

// Rows rc at a time, from the LDS left by the columns: as many workgroups per
// CU as their registers allow (20 waves in single precision, 12 in FP64), fewer
// where a pass over rc rows would then leave most threads idle.  N = 72 in
// single precision, alone: 36 rows (35 KB) 134 us per 128 bands, 7 rows (26 KB) 276;
// N = 160, 64 band pairs: 80 rows 819 us, 14 rows 1 480.
bool rows_geometry(bool f64, int n, int ext, bool tight, TwoGeom *g) {
  const int b = plane2::factor_b(n), a = n / b, nt = plane2::threads(f64, n);
  const size_t cs = f64 ? 16 : 8;
  g->tight = tight;
  g->b = b;
  g->bp = tight ? b : plane2::pitch_b(b);
  g->ldT = tight ? n | 1 : plane2::pitch(n, b);
  const size_t tile = cs * (size_t)ext * g->ldT;
  const size_t per_row = cs * (size_t)(a - ext / b) * b;   // extra slots of a row
  for (int wg = std::max(1, (f64 ? 12 : 20) * 64 / nt + (f64 && nt == 512)); wg >= 1; --wg) {
    const size_t cap = (size_t)kLdsMax / wg;
    if (tile >= cap) continue;
    int rc = per_row ? (int)std::min<size_t>(n, (cap - tile) / per_row) : n;
    while (rc > 0 && tile + per_row * (rc | 1) > cap) --rc;
    if (rc == 0 || (wg > 1 && rc < n && 5 * rc * b < 2 * nt)) continue;
    const int chunks = (n + rc - 1) / rc;
    g->rc = (n + chunks - 1) / chunks;
    g->lds = tile + per_row * (g->rc | 1);
    return true;
  }
  return false;
}

}  // namespace

// Where the columns leave room for a few rows only, a row pass employs few of
// the threads (rc b items for nt) between its barriers.  Then the unpadded columns
// are taken where they are compiled and the padded ones employ less than a sixth.
// The LDS-pass kernel is the faster one where a pass employs less than 1/18 of the
// threads, the split kernel where less than 1/12.  Per launch of 24 planes (us), FP64
// (32 bands), two-factor and the kernel instead of it (s: split):
//   N = 128  65 columns, 11 rows 153, 252    68, 5 rows 247, 313    69, 3 rows  357, 314
//       144  62 columns, 5 rows  257, 499    63, 3 rows 390, 558    64, 1 row  1167, 662
//       140  63 columns, 5 rows  273, 362    64, 3 rows 420, 410
//       135  72 columns, 7 rows  214, 2011   73, 5 rows 304, 305s   74, 3 rows  455, 302s
// single precision (64 bands), padded, unpadded and the kernel instead of both
// (-: does not fit), the lane octets that the two-factor kernel replaced (*):
//   N = 144  127 columns 262, 211, 761, 300*   129 398, 214, 788, 310*
//            135 -, 239, 1605, 327*   140 -, 331, 568s
//       160  109 columns 272, 206, 531, 289*   113 423, 221, 618, 297*
//            121 -, 268, 1571, 311*   123 -, 340, 4281, 317*   125 -, 529, 540s
//       192  89 columns 293, 252, 644   95 697, 314, 850   103 -, 796, 593s
// split: whether the split kernel, not the LDS-pass one, would run instead.
bool two_geometry(int prec, int n1, int n2, int ext, int exty, bool split, TwoGeom *g) {
  *g = TwoGeom{};
  if (n1 != n2) return false;
  switch (n1) {
#define QEH_TWO_CASE(NN) case NN:
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    break;
    default: return false;
  }
  const bool f64 = prec == QEH_FP64;
  const int n = n1, b = plane2::factor_b(n), nt = plane2::threads(f64, n);
  bool ok = rows_geometry(f64, n, ext, false, g);
  if (plane2::has_tight(f64, n) && (!ok || 6 * g->rc * b < nt)) {
    TwoGeom t{};
    if (rows_geometry(f64, n, ext, true, &t) && t.rc > g->rc) {
      *g = t;
      ok = true;
    }
  }
  if (!ok || (g->rc < n && (split ? 12 : 18) * g->rc * b < nt)) {
    *g = TwoGeom{};
    return false;
  }
  g->half = std::max(ext, exty) <= (n / b + 1) / 2 * b ? 1 : 0;
  g->on = 1;
  return true;
}

hipError_t launch_density_two_f32(const qeh_ctx *c, int nbk, int bsub, const double *occ,
                                  double *partial) {
  switch (c->n1) {
#define QEH_TWO_CASE(NN) \
  case NN: return plane2::launch_density<float2, NN>(c, nbk, bsub, occ, partial);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return hipErrorInvalidValue;
  }
}

size_t density_two_lds_f32(int n, int ext) {
  switch (n) {
#define QEH_TWO_CASE(NN) \
  case NN: return plane2::density_lds<float2, NN>(ext);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return 0;
  }
}

}  // namespace qeh
