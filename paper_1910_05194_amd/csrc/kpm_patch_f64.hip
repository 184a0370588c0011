// Patch kernels in FP64 (kpm_patch.h).
#include "kpm_patch.h"

namespace kpm {

void* patch_fn_f64(int kind, bool phase, int spt, bool hist) {
  return hist ? pick_patch_kind<double, true>(kind, phase, spt) : pick_patch_kind<double, false>(kind, phase, spt);
}

}  // namespace kpm
