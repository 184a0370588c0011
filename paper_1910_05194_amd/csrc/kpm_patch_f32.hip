// Patch kernels in FP32 (kpm_patch.h).
#include "kpm_patch.h"

namespace kpm {

void* patch_fn_f32(int kind, bool phase, int spt, bool hist) {
  return hist ? pick_patch_kind<float, true>(kind, phase, spt) : pick_patch_kind<float, false>(kind, phase, spt);
}

}  // namespace kpm
