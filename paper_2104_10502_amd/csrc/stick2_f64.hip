// Two-factor z transforms, double precision (see stick2.h).
#include "stick2.h"

namespace qeh {

hipError_t launch_k1_two_f64(const qeh_ctx *c, int np, const double2 *psi, int ldpsi, int nbk,
                             const int2 *pairs, float2 *psi32) {
  switch (c->n3) {
#define QEH_TWO_CASE(NN) \
  case NN: return stick2::launch_k1<double2, NN>(c, np, psi, ldpsi, nbk, pairs, psi32);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_k3_two_f64(const qeh_ctx *c, int nbk, const double2 *psi, int ldpsi,
                             double2 *hpsi, int ldh) {
  switch (c->n3) {
#define QEH_TWO_CASE(NN) \
  case NN: return stick2::launch_k3<double2, NN>(c, nbk, psi, ldpsi, hpsi, ldh);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qeh
