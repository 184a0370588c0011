// Patch kernels (kpm_patch.h): choice of the shape, launches.
#include "kpm_patch.h"

#include <algorithm>

namespace kpm {

void* patch_fn_f32(int kind, bool phase, int spt, bool hist);
void* patch_fn_f64(int kind, bool phase, int spt, bool hist);

// Modelled time of one step (us) with n patches per CU: a launch of 5, and per patch
// the loads, the reduction and ks steps, scaled by what a site costs.  Measured
// launches (us), honeycomb FP32, one patch per CU: 1 site per thread 7.1 (4 steps),
// 8.0 (6); 2 sites 9.4 (8); 4 sites 9.6 (4), 12.6 (8); 4 sites and 8 steps with 2 and
// 3.3 patches per CU 25 and 36.  FP64 with phases takes 1.8 times as much per patch,
// a spin 1.7 in FP32 and 3 in FP64.  mem_us: the vectors in and out, not hidden in a
// launch of one or two rounds.
static double patch_time(const kpm_plan* P, int spt, int ks, int n, double mem_us) {
  double g = P->n_spin == 2 ? 1.7 : 1.0;
  if (P->prec == KPM_FP64) g *= P->n_spin == 2 ? 1.8 : 1.1;
  if (P->has_phase) g *= P->prec == KPM_FP64 && P->n_spin == 1 ? 1.7 : 1.2;
  return (5.0 + mem_us + n * g * (0.6 * spt + ks * (0.35 + 0.1 * spt))) / ks;
}

bool patch_shape(const kpm_plan* P, bool hist, int max_steps, int lds_max, int n_cu, PatchShape* best) {
  *best = PatchShape();
  const int n_lat = (int)P->lats.size();
  int max_l1 = 0;
  double cells = 0.0;
  for (const kpm_lattice_t& L : P->lats) {
    max_l1 = std::max(max_l1, L.L1);
    cells += (double)L.L1 * L.L2;
    // 32-bit element offsets within a lattice's block.
    if ((double)L.L1 * L.L2 * P->n_sub * P->n_spin * P->Rp * 2.0 >= 2147483648.0) return false;
  }
  const int max_tiles = std::min(2048, kPatchRounds * n_cu);
  double best_t = 1e30;
  const double vec_us = (double)P->n_orb * P->Rp * 2 * P->tsize / 5.0e6;
  const int ks_max = std::min(max_steps, patch_steps(P->kind));
  for (int lgw = 0; lgw <= 3 && (1 << lgw) < 2 * P->E; ++lgw) {
    const int n_rg = (int)ceil_div(P->E, 1 << lgw);
    for (int spt = 1; spt <= 4; spt <<= 1) {
      const int cap = kPatchBlock * spt / (P->n_sub << lgw);   // cells
      for (int ks = 2; ks <= ks_max; ++ks) {
        for (int bx = 1; bx <= 64 && bx <= max_l1; ++bx) {
          const int px = (int)ceil_div(max_l1, bx), ex = px + 2 * ks;
          const int py = cap / ex - 2 * ks;
          if (py < 1) continue;
          if (cells * n_rg / ((double)px * py) > max_tiles) continue;
          const size_t lds = 2 * (size_t)P->n_spin * (kPatchBlock * spt + 2 * (ex + 1) * (P->n_sub << lgw)) * 16;
          if (lds > (size_t)lds_max) continue;
          int64_t tiles = 0;
          for (int l = 0; l < n_lat; ++l) tiles += n_rg * ceil_div(P->lats[l].L1, px) * ceil_div(P->lats[l].L2, py);
          if (tiles > max_tiles) continue;
          // Two vectors come in with their halos, two (or one per step) go out, at 5 TB/s.
          const double mem_us = vec_us * (2.0 * (double)tiles * ex * (py + 2 * ks) / (cells * n_rg) + (hist ? ks : 2));
          const double t = patch_time(P, spt, ks, (int)ceil_div(tiles, n_cu), mem_us);
          if (t < best_t) {
            best_t = t;
            best->px = px;
            best->py = py;
            best->ks = ks;
            best->ex = ex;
            best->spt = spt;
            best->lgw = lgw;
            best->lds_bytes = lds;
            best->us_per_step = t;
          }
        }
      }
    }
  }
  if (best->ks == 0) return false;
  best->fn = P->prec == KPM_FP32 ? patch_fn_f32(P->kind, P->has_phase, best->spt, hist)
                                 : patch_fn_f64(P->kind, P->has_phase, best->spt, hist);
  return true;
}

template <typename T>
static hipError_t launch_patch(const kpm_plan* P, const PatchShape& S, hipStream_t s, const int4* tiles,
                               const int* slot_of, int n_tiles, const void* v, const void* w, int nlev,
                               void* const* out, double* part, int64_t part_stride) {
  PatchArgs<T> a = {};
  a.lats = (const LatDev<T>*)P->latdev;
  a.tiles = tiles;
  a.slot_of = slot_of;
  a.n_tiles = n_tiles;
  a.v = (const T*)v;
  a.w = (const T*)(w ? w : v);
  a.onsite = P->has_onsite ? (const T*)P->onsite : nullptr;
  a.mask = P->has_mask ? P->mask : nullptr;
  a.phase = (const T*)P->phase;
  for (int l = 0; l < kPatchSteps; ++l) a.out[l] = (T*)out[part ? std::min(l, 1) : std::min(l, nlev - 1)];
  a.part = part;
  a.part_stride = part_stride;
  a.a1 = w ? (T)2 : (T)1;
  a.b1 = w ? (T)1 : (T)0;
  a.read_w1 = w ? 1 : 0;
  a.nlev = nlev;
  a.px = S.px;
  a.py = S.py;
  a.ks = S.ks;
  a.ex = S.ex;
  a.inv_ex = 1.0f / (float)S.ex;
  a.cells = S.ex * (S.py + 2 * S.ks);
  a.E = P->E;
  a.lgw = S.lgw;
  a.Rp = P->Rp;
  void* args[] = {&a};
  return after_call(hipLaunchKernel(S.fn, dim3((unsigned)(ceil_div(n_tiles, 8) * 8)), dim3(kPatchBlock), args,
                                    S.lds_bytes, s));
}

hipError_t patch_run(const kpm_plan* P, const PatchShape& S, hipStream_t s, const int4* tiles, const int* slot_of,
                     int n_tiles, const void* v, const void* w, int nlev, void* const* out, double* part,
                     int64_t part_stride) {
  if (nlev < 1 || nlev > S.ks) return hipErrorInvalidValue;
  count_launch(kLaunchPatch);
  return P->prec == KPM_FP32
             ? launch_patch<float>(P, S, s, tiles, slot_of, n_tiles, v, w, nlev, out, part, part_stride)
             : launch_patch<double>(P, S, s, tiles, slot_of, n_tiles, v, w, nlev, out, part, part_stride);
}

}  // namespace kpm
