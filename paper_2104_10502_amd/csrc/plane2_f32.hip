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

// Rows rc at a time, from the LDS left by the columns: as many workgroups per
// CU as their registers allow (20 waves in single precision, 12 in FP64), fewer
// where a pass over rc rows would then leave most threads idle.  N = 72 in
// single precision: 36 rows (35 KB) 134 us per 128 bands, 7 rows (26 KB) 276;
// N = 160: 80 rows 819 us, 14 rows 1 480.
bool two_geometry(int prec, int n1, int n2, int ext, int exty, TwoGeom *g) {
  g->on = 0;
  g->half = 0;
  g->rc = 0;
  g->lds = 0;
  if (n1 != n2) return false;
  switch (n1) {
#define QEH_TWO_CASE(NN) case NN:
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    break;
    default: return false;
  }
  const bool f64 = prec == QEH_FP64;
  const int n = n1, b = plane2::factor_b(n), a = n / b, nt = plane2::threads(f64, n);
  const size_t cs = f64 ? 16 : 8;
  const size_t tile = cs * (size_t)ext * plane2::pitch(n, b);
  const size_t per_row = cs * (size_t)(a - ext / b) * b;   // extra slots of a row
  g->ldT = plane2::pitch(n, b);
  g->bp = plane2::pitch_b(b);
  g->b = b;
  g->half = std::max(ext, exty) <= (a + 1) / 2 * b ? 1 : 0;
  for (int wg = std::max(1, (f64 ? 12 : 20) * 64 / nt + (f64 && nt == 512)); wg >= 1; --wg) {
    const size_t cap = (size_t)kLdsMax / wg;
    if (tile >= cap) continue;
    int rc = per_row ? (int)std::min<size_t>(n, (cap - tile) / per_row) : n;
    while (rc > 0 && tile + per_row * (rc | 1) > cap) --rc;
    if (rc == 0 || (wg > 1 && rc < n && 5 * rc * b < 2 * nt)) continue;
    const int chunks = (n + rc - 1) / rc;
    g->rc = (n + chunks - 1) / chunks;
    g->lds = tile + per_row * (g->rc | 1);
    g->on = 1;
    return true;
  }
  return false;
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
