// Patches of the conductivity chains on small spinless lattices: the layout of
// kpm_patch.h, the site arithmetic and the stores of the chain sweeps.  Level l of a
// launch writes one Gamma block row: its value (mode 0, L chain) or the velocity of the
// level below it (mode 1, R chain), and the last two levels go back to HBM.  Every item
// keeps its column's coefficients in registers.
#include "kpm_chain.h"
#include "kpm_plan.h"

namespace kpm {

template <typename T>
struct PatchChainArgs {
  const LatDev<T>* __restrict__ lats;
  const int4* __restrict__ tiles;
  int n_tiles;
  const T* __restrict__ v;
  const T* __restrict__ w;
  const T* __restrict__ onsite;      // or nullptr
  const uint8_t* __restrict__ mask;  // or nullptr
  const T* __restrict__ phase;       // or nullptr
  T* out_a;                          // level nlev - 1 (nlev >= 2)
  T* out_b;                          // level nlev
  T* blk;
  __bf16* blk_lo;
  int64_t blk_row0, blk_rows;
  T a1, b1, vel_scale;
  int read_w1, nlev, vdir;
  int px, py, ks, ex, cells;
  float inv_ex;
  int E, lgw, Rp;
};

template <typename T, int KIND, int SPT, int MODE, bool SPLIT>
__global__ void __launch_bounds__(kPatchBlock) patch_chain_kernel(PatchChainArgs<T> A) {
  using P = Pack<T>;
  constexpr int NC = P::NC;
  constexpr int NSUB = KindTraits<KIND>::NSUB;
  constexpr int NNB = KindTraits<KIND>::NNB;
  constexpr int LGS = NSUB == 2 ? 1 : 0;
  static_assert(KindTraits<KIND>::NSPIN == 1 && (!SPLIT || sizeof(T) == 4), "spinless; split BF16 stores FP32 values");
  extern __shared__ double lds[];
  const int t0 = (int)(((int64_t)(blockIdx.x & 7) * A.n_tiles) >> 3);
  const int t1 = (int)(((int64_t)((blockIdx.x & 7) + 1) * A.n_tiles) >> 3);
  const int ti = t0 + (int)(blockIdx.x >> 3);
  if (ti >= t1) return;
  const int tid = threadIdx.x;
  const int4 tl = A.tiles[ti];
  const LatDev<T>& Lg = A.lats[tl.x];
  const int L1 = Lg.L1, L2 = Lg.L2;
  const int lgw = A.lgw, ew = 1 << lgw;
  const int s = (tid >> lgw) & (NSUB - 1);
  const int c = tl.y * ew + (tid & (ew - 1));
  const int halo = A.ks, ex = A.ex;
  const int nx = min(A.px, L1 - tl.z), ny = min(A.py, L2 - tl.w);

  P v[SPT], w[SPT];
  T ons[SPT];
  bool alive[SPT], inner[SPT];
  uint32_t off[SPT];
  Coef<T, KIND> C[SPT];
#pragma unroll
  for (int k = 0; k < SPT; ++k) {
    const int cell = (tid + k * kPatchBlock) >> (lgw + LGS);
    const int cy = (int)(((float)cell + 0.5f) * A.inv_ex), cx = cell - cy * ex;   // exact: cell < 4096
    const bool ok = cell < A.cells && c < A.E;
    int x = tl.z - halo + cx, y = tl.w - halo + cy;
    while (x < 0) x += L1;
    while (x >= L1) x -= L1;
    while (y < 0) y += L2;
    while (y >= L2) y -= L2;
    inner[k] = ok && (uint32_t)(cx - halo) < (uint32_t)nx && (uint32_t)(cy - halo) < (uint32_t)ny;
    const uint32_t site = ok ? (uint32_t)((y * L1 + x) * NSUB + s) : 0u;
    off[k] = (site * (uint32_t)A.Rp + (ok ? (uint32_t)c * NC : 0u)) * 2;
    v[k] = ld_pack(A.v + Lg.vec_off + off[k]);
    w[k] = ld_pack(A.w + Lg.vec_off + off[k]);
    ons[k] = A.onsite ? A.onsite[Lg.site_off + site] : Lg.onsite_const;
    alive[k] = A.mask ? A.mask[Lg.site_off + site] != 0 : true;
    const int n1 = ok ? x : 0, n1m = n1 == 0 ? L1 - 1 : n1 - 1;
#pragma unroll
    for (int b = 0; b < NNB; ++b) {
      T pre = 1, pim = 0;
      if (KIND != KPM_SQUARE && A.phase) {
        const T* ph = A.phase + 2 * (Lg.phase_off + (int64_t)((s == 0 || b != 1) ? n1 : n1m) * 3 + b);
        pre = ph[0];
        pim = s == 0 ? ph[1] : -ph[1];
      }
      C[k].re[b][0] = Lg.hop * pre;
      C[k].im[b][0] = Lg.hop * pim;
      C[k].vc[b] = MODE == 1 ? Lg.vc[A.vdir][s][b] : (T)0;
    }
  }
  const int cw = NSUB << lgw;
  const int guard = (ex + 1) * cw;
  const int plane = SPT * kPatchBlock + 2 * guard;
  P* cur = reinterpret_cast<P*>(lds) + guard + tid;
  P* nxt = cur + plane;
  int nb[NNB];
  if constexpr (KIND == KPM_SQUARE) {
    nb[0] = cw;
    nb[1] = -cw;
    nb[2] = ex * cw;
    nb[3] = -ex * cw;
  } else {
    const int o = s == 0 ? ew : -ew;
    nb[0] = o;
    nb[1] = s == 0 ? o - (ex - 1) * cw : o + (ex - 1) * cw;
    nb[2] = s == 0 ? o - ex * cw : o + ex * cw;
  }
#pragma unroll
  for (int k = 0; k < SPT; ++k) cur[k * kPatchBlock] = v[k];
  __syncthreads();
#pragma unroll 1
  for (int l = 0; l < A.nlev; ++l) {
    const T a = l == 0 ? A.a1 : (T)2, b = l == 0 ? A.b1 : (T)1;
    const bool rw = l > 0 || A.read_w1 != 0;
    const int64_t brow = A.blk_row0 + l + (MODE == 0 ? 1 : 0);
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
      P vn[NNB][1], o, g = {};
#pragma unroll
      for (int q = 0; q < NNB; ++q) vn[q][0] = cur[k * kPatchBlock + nb[q]];
      chain_site<T, KIND, MODE>(a, b, rw, C[k], ons[k], A.vel_scale, alive[k], v[k], w[k], vn, o, g);
      w[k] = v[k];
      v[k] = o;
      nxt[k * kPatchBlock] = o;
      if (inner[k]) {
        // NC complex values of one K block (the block is a multiple of a pack).
        const int64_t e = (Lg.vec_off + off[k]) / 2;
        const int64_t at = 2 * ((e / kBlkK) * A.blk_rows * kBlkK + brow * kBlkK + e % kBlkK);
        const P src = MODE == 0 ? o : g;
        if constexpr (SPLIT) {
          typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
          bf16x4 hi, lo;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            hi[q] = (__bf16)src.v[q];
            lo[q] = (__bf16)((float)src.v[q] - (float)hi[q]);
          }
          *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(A.blk) + at) = hi;
          *reinterpret_cast<bf16x4*>(A.blk_lo + at) = lo;
        } else {
          st_pack(A.blk + at, src);
        }
      }
    }
    P* t = cur;
    cur = nxt;
    nxt = t;
    lds_barrier();
  }
#pragma unroll
  for (int k = 0; k < SPT; ++k) {
    if (inner[k]) {
      st_pack(A.out_b + Lg.vec_off + off[k], v[k]);
      if (A.nlev >= 2) st_pack(A.out_a + Lg.vec_off + off[k], w[k]);
    }
  }
}

template <typename T, int KIND, int SPT>
static void* pick_mode(int mode, bool split) {
  if constexpr (sizeof(T) == 4) {
    if (split)
      return mode == 0 ? (void*)patch_chain_kernel<T, KIND, SPT, 0, true> : (void*)patch_chain_kernel<T, KIND, SPT, 1, true>;
  }
  return mode == 0 ? (void*)patch_chain_kernel<T, KIND, SPT, 0, false> : (void*)patch_chain_kernel<T, KIND, SPT, 1, false>;
}
template <typename T, int KIND>
static void* pick_spt(int spt, int mode, bool split) {
  if (spt == 1) return pick_mode<T, KIND, 1>(mode, split);
  if (spt == 2) return pick_mode<T, KIND, 2>(mode, split);
  return pick_mode<T, KIND, 4>(mode, split);
}

void* patch_chain_fn(int prec, int kind, int spt, int mode, bool split) {
  if (kind == KPM_HONEYCOMB_SPIN || (mode != 0 && mode != 1) || (split && prec != KPM_FP32)) return nullptr;
  if (prec == KPM_FP32)
    return kind == KPM_SQUARE ? pick_spt<float, KPM_SQUARE>(spt, mode, split) : pick_spt<float, KPM_HONEYCOMB>(spt, mode, split);
  return kind == KPM_SQUARE ? pick_spt<double, KPM_SQUARE>(spt, mode, false) : pick_spt<double, KPM_HONEYCOMB>(spt, mode, false);
}

template <typename T>
static hipError_t launch(const kpm_plan* P, const ChainPlan& C, hipStream_t s, int mode, const void* v, const void* w,
                         void* out_a, void* out_b, bool first, int nlev, void* blk, void* blk_lo, int64_t row0,
                         int64_t blk_rows, int vdir, double vel_scale) {
  const PatchShape& S = C.patch;
  PatchChainArgs<T> a = {};
  a.lats = (const LatDev<T>*)P->latdev;
  a.tiles = C.tiles;
  a.n_tiles = C.n_tiles;
  a.v = (const T*)v;
  a.w = (const T*)(first ? v : w);
  a.onsite = P->has_onsite ? (const T*)P->onsite : nullptr;
  a.mask = P->has_mask ? P->mask : nullptr;
  a.phase = P->has_phase ? (const T*)P->phase : nullptr;
  a.out_a = (T*)out_a;
  a.out_b = (T*)out_b;
  a.blk = (T*)blk;
  a.blk_lo = (__bf16*)blk_lo;
  a.blk_row0 = row0;
  a.blk_rows = blk_rows;
  a.a1 = first ? (T)1 : (T)2;
  a.b1 = first ? (T)0 : (T)1;
  a.vel_scale = (T)vel_scale;
  a.read_w1 = first ? 0 : 1;
  a.nlev = nlev;
  a.vdir = vdir;
  a.px = S.px;
  a.py = S.py;
  a.ks = S.ks;
  a.ex = S.ex;
  a.cells = S.ex * (S.py + 2 * S.ks);
  a.inv_ex = 1.0f / (float)S.ex;
  a.E = P->E;
  a.lgw = S.lgw;
  a.Rp = P->Rp;
  void* args[] = {&a};
  void* fn = C.fn[mode][blk_lo != nullptr ? 1 : 0];
  if (fn == nullptr || nlev < 1 || nlev > S.ks) return hipErrorInvalidValue;
  count_launch(kLaunchPatchChain);
  return after_call(hipLaunchKernel(fn, dim3((unsigned)(ceil_div(C.n_tiles, 8) * 8)), dim3(kPatchBlock), args, S.lds_bytes, s));
}

hipError_t patch_chain_run(const kpm_plan* P, const ChainPlan& C, hipStream_t s, int mode, const void* v, const void* w,
                           void* out_a, void* out_b, bool first, int nlev, void* blk, void* blk_lo, int64_t row0,
                           int64_t blk_rows, int vdir, double vel_scale) {
  return P->prec == KPM_FP32 ? launch<float>(P, C, s, mode, v, w, out_a, out_b, first, nlev, blk, blk_lo, row0, blk_rows, vdir, vel_scale)
                             : launch<double>(P, C, s, mode, v, w, out_a, out_b, first, nlev, blk, blk_lo, row0, blk_rows, vdir, vel_scale);
}

}  // namespace kpm
