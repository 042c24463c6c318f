// Resident-value kernels of dense BF16 / FP8 tables.

#include "mbdp_resident.h"

namespace mbdp {

SolveFn pick_resident_lp(const KParams& p, ResShape shape) {
  if (p.vdtype == kBF16) return resident_fn<ValBF16, false>(shape, p.task);
  if (p.vdtype == kFP8) return resident_fn<ValFP8, false>(shape, p.task);
  return nullptr;
}

}  // namespace mbdp
