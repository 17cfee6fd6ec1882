// Two-factor z transforms, single precision (see stick2.h).
#include "stick2.h"

namespace qeh {

hipError_t launch_k1_two_f32(const qeh_ctx *c, int np, const double2 *psi, int ldpsi, int nbk,
                             const int2 *pairs, float2 *psi32) {
  switch (c->n3) {
#define QEH_TWO_CASE(NN) \
  case NN: return stick2::launch_k1<float2, NN>(c, np, psi, ldpsi, nbk, pairs, psi32);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_k3_two_f32(const qeh_ctx *c, int nbk, const double2 *psi, int ldpsi,
                             double2 *hpsi, int ldh) {
  switch (c->n3) {
#define QEH_TWO_CASE(NN) \
  case NN: return stick2::launch_k3<float2, NN>(c, nbk, psi, ldpsi, hpsi, ldh);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return hipErrorInvalidValue;
  }
}

// 16 sticks a workgroup in FP64, 32 in single precision: rows of 256 bytes and,
// up to about 100 points, five or more workgroups' lines in a CU's LDS (FP64, K1 / K3
// of 72 points, 128 bands: 8 sticks 47 / 54 us, 16 40 / 46, 32 47 / 46; single precision
// of 168 points, 64 Gamma pairs: 16 190 / 124, 32 190 / 103, 64 345 / 181, before
// the mirror images).
bool stick_two_geometry(int prec, int n3, int lmin, int lmax, StickTwoGeom *g) {
  g->on = 0;
  switch (n3) {
#define QEH_TWO_CASE(NN) case NN:
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    break;
    default: return false;
  }
  const bool f64 = prec == QEH_FP64;
  const int b = plane2::factor_b(n3), a = n3 / b;
  g->b = b;
  g->bp = plane2::pitch_b(b);
  g->ldz = plane2::pitch(n3, b);
  g->half = lmax < stick2::low_values(a) * b && -lmin <= stick2::high_values(a) * b;
  g->sl = f64 ? 4 : 5;
  g->lds = (f64 ? 16 : 8) * ((size_t)n3 + ((size_t)g->ldz << g->sl));
  g->on = 1;
  return true;
}

}  // namespace qeh
