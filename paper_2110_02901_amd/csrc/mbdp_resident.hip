// Resident-value kernels of dense FP32 tables.

#include "mbdp_resident.h"

namespace mbdp {

SolveFn pick_resident(const KParams& p, ResShape shape) {
  return p.n % 4 ? resident_fn<ValF32, true>(shape, p.task) : resident_fn<ValF32, false>(shape, p.task);
}

}  // namespace mbdp
