// Two-factor plane pass, double precision (see plane2.h).
#include "plane2.h"

namespace qeh {

hipError_t launch_k2_two_f64(const qeh_ctx *c, int nbk) {
  switch (c->n1) {
#define QEH_TWO_CASE(NN) \
  case NN: return plane2::launch<double2, NN>(c, nbk);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_density_two_f64(const qeh_ctx *c, int nbk, int bsub, const double *occ,
                                  double *partial) {
  switch (c->n1) {
#define QEH_TWO_CASE(NN) \
  case NN: return plane2::launch_density<double2, NN>(c, nbk, bsub, occ, partial);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return hipErrorInvalidValue;
  }
}

size_t density_two_lds_f64(int n, int ext) {
  switch (n) {
#define QEH_TWO_CASE(NN) \
  case NN: return plane2::density_lds<double2, NN>(ext);
    QEH_TWO_SIZES(QEH_TWO_CASE)
#undef QEH_TWO_CASE
    default: return 0;
  }
}

}  // namespace qeh
