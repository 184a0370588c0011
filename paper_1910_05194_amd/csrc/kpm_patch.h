// Patch kernels: several recursion steps per launch on lattices too small to fill
// the chip with rows.
//
// A workgroup takes a patch of PX x PY cells of one lattice with a halo of KS cells
// on each side, for Ew 16-byte chunks of the vectors.  The patch's v_n sits in LDS
// (two buffers, one barrier per step), every thread keeps its own sites' v_n and
// v_{n-1} in registers, and KS steps run before the result leaves the workgroup:
// after l of them the cells at a distance of l or more from the patch's edge are
// right, after KS the interior.
//
// What bounds it is latency: a launch costs about 5 us whatever it does, a step 0.4
// to 0.7 us of LDS round trips, dependent FMAs and one barrier (with a spin the FMAs
// themselves).  The row-streaming sweep pays 3 KS - 3 rows of skew per tile at about
// 1.25 us a row, the single-step kernels a launch per step; the patch pays halo cells
// instead, (PX + 2 KS)(PY + 2 KS) for PX PY.  Per step (us), before -> patches:
// honeycomb 64 x 64, 4 vectors, FP64 4.08 -> 1.5; 128 x 128, 4, FP32 4.95 -> 1.9;
// square 273 x 197, 8, FP64 5.5 -> 4.0; spinful 64 x 64, 4, FP32 5.7 -> 2.2;
// 164 x 142, 2 7.1 -> 2.8; 512 x 512, 8 vectors would be 35 -> 52 (rows stay).
// Workgroups of 1024 threads with half the sites each: 5 to 15 % slower.
//
// Items: one site's chunk (both spins).  Item i = cell * (NSUB Ew) + s Ew + cl is
// thread i % 512's item i / 512, at LDS pack i, so neighbours are fixed offsets and
// all lanes of an access are contiguous.  A neighbour of an edge cell may be any
// other item or the guard space before and after the buffer: only values that the
// shrinking region has already given up depend on it.
#pragma once

#include "kpm_plan.h"
#include "kpm_stencil.h"

namespace kpm {

// A site's hopping constants: the amplitude, on the spin lattice the 2 x 2 blocks
// as sublattice s meets them (B: the conjugate transpose).
template <typename T, int KIND>
struct SiteCoef {
  T hop;
};
template <typename T>
struct SiteCoef<T, KPM_HONEYCOMB_SPIN> {
  T hop, exch;
  T re[3][2][2], im[3][2][2];
};
template <typename T, int KIND>
__device__ inline void site_coef(const LatDev<T>& L, int s, SiteCoef<T, KIND>& C) {
  C.hop = L.hop;
  if constexpr (KIND == KPM_HONEYCOMB_SPIN) {
    C.exch = L.exch;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          C.re[k][p][q] = s == 0 ? L.blk[k][2 * (2 * p + q)] : L.blk[k][2 * (2 * q + p)];
          C.im[k][p][q] = s == 0 ? L.blk[k][2 * (2 * p + q) + 1] : -L.blk[k][2 * (2 * q + p) + 1];
        }
  }
}

// One step at one site, in the arithmetic of the kernels that serve larger lattices
// (sweeps without a spin, single steps with one): the vectors are the same to the bit.
template <typename T, int KIND, bool PHASE, bool HIST>
__device__ inline void site_step(T a, T b, bool read_w, const SiteCoef<T, KIND>& C, const T* hre, const T* him, T ons,
                                 bool alive, const Pack<T> (&vo)[KindTraits<KIND>::NSPIN],
                                 const Pack<T> (&wo)[KindTraits<KIND>::NSPIN],
                                 const Pack<T> (&vn)[KindTraits<KIND>::NNB][KindTraits<KIND>::NSPIN],
                                 Pack<T> (&out)[KindTraits<KIND>::NSPIN], bool acc, double* pv, double* pw) {
  constexpr int NC = Pack<T>::NC;
  if constexpr (KIND != KPM_HONEYCOMB_SPIN) {
    Pack<T> n[KindTraits<KIND>::NNB];
#pragma unroll
    for (int k = 0; k < KindTraits<KIND>::NNB; ++k) n[k] = vn[k][0];
    sweep_site<T, KIND, PHASE, HIST>(a, b, read_w, C.hop, hre, him, ons, alive, vo[0], wo[0], n, out[0], acc, pv, pw);
  } else {
#pragma unroll
    for (int sp = 0; sp < 2; ++sp) {
      const T onsp = ons + (sp == 0 ? C.exch : -C.exch);
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        T hr = onsp * vo[sp].v[2 * j], hi = onsp * vo[sp].v[2 * j + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          T tr = 0, ti = 0, br = 0, bi = 0;
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2)
            cmul_acc(br, bi, C.re[k][sp][s2], C.im[k][sp][s2], vn[k][s2].v[2 * j], vn[k][s2].v[2 * j + 1]);
          if constexpr (PHASE) cmul_acc(tr, ti, hre[k], him[k], br, bi);
          else { tr = br; ti = bi; }
          hr += tr;
          hi += ti;
        }
        T orr = a * hr, oi = a * hi;
        if (read_w) {
          orr -= b * wo[sp].v[2 * j];
          oi -= b * wo[sp].v[2 * j + 1];
        }
        if (!alive) {
          orr = 0;
          oi = 0;
        }
        out[sp].v[2 * j] = orr;
        out[sp].v[2 * j + 1] = oi;
      }
    }
    if (!HIST && acc) {
#pragma unroll
      for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int j = 0; j < NC; ++j) {
          const double xr = vo[sp].v[2 * j], xi = vo[sp].v[2 * j + 1];
          pv[j] = fma(xr, xr, fma(xi, xi, pv[j]));
          pw[j] = fma((double)out[sp].v[2 * j], xr, fma((double)out[sp].v[2 * j + 1], xi, pw[j]));
        }
    }
  }
}

template <typename T>
struct PatchArgs {
  const LatDev<T>* __restrict__ lats;
  const int4* __restrict__ tiles;   // (lattice, r-group, x0, y0), the first interior cell
  const int* __restrict__ slot_of;
  int n_tiles;
  const T* __restrict__ v;          // v_n
  const T* __restrict__ w;          // v_{n-1} (read when read_w1)
  const T* __restrict__ onsite;     // or nullptr
  const uint8_t* __restrict__ mask; // or nullptr
  const T* __restrict__ phase;
  T* out[kPatchSteps];              // HIST: levels 1 .. nlev; else [0] = v_{n+nlev-1} (nlev >= 2), [1] = v_{n+nlev}
  double* part;                     // slot partials of step n (not HIST), part_stride doubles per step
  int64_t part_stride;
  T a1, b1;
  int read_w1, nlev;
  int px, py, ks, ex, cells;        // interior, halo, thread cells per row and in all
  float inv_ex;
  int E, lgw, Rp;                   // chunks, log2 of the chunks per patch
};

// HIST: every level goes to HBM and no products are formed (see the history sweeps).
template <typename T, int KIND, bool PHASE, int SPT, bool HIST>
__global__ void __launch_bounds__(kPatchBlock) patch_kernel(PatchArgs<T> A) {
  using P = Pack<T>;
  constexpr int NC = P::NC;
  constexpr int NSUB = KindTraits<KIND>::NSUB;
  constexpr int NSPIN = KindTraits<KIND>::NSPIN;
  constexpr int NNB = KindTraits<KIND>::NNB;
  constexpr int LGS = NSUB == 2 ? 1 : 0;
  constexpr int KS = patch_steps(KIND);
  extern __shared__ double lds[];

  // XCD-aware: workgroup b runs on XCD b % 8, which owns a contiguous range of tiles.
  const int t0 = (int)(((int64_t)(blockIdx.x & 7) * A.n_tiles) >> 3);
  const int t1 = (int)(((int64_t)((blockIdx.x & 7) + 1) * A.n_tiles) >> 3);
  const int ti = t0 + (int)(blockIdx.x >> 3);
  if (ti >= t1) return;
  const int tid = threadIdx.x;
  const int4 tl = A.tiles[ti];
  const LatDev<T>& Lg = A.lats[tl.x];
  const int L1 = Lg.L1, L2 = Lg.L2;
  const int lgw = A.lgw, ew = 1 << lgw;
  const int cl = tid & (ew - 1);
  const int s = (tid >> lgw) & (NSUB - 1);
  const int c = tl.y * ew + cl;
  const int halo = A.ks, ex = A.ex;
  const int nx = min(A.px, L1 - tl.z), ny = min(A.py, L2 - tl.w);
  SiteCoef<T, KIND> C;
  site_coef<T, KIND>(Lg, s, C);

  // Every item loads from its site; surplus items (beyond the patch or the chunks)
  // from the lattice's first site.
  P v[SPT][NSPIN], w[SPT][NSPIN];
  T ons[SPT];
  bool alive[SPT], inner[SPT];
  uint32_t off[SPT];
  int col[SPT];
#pragma unroll
  for (int k = 0; k < SPT; ++k) {
    const int cell = (tid + k * kPatchBlock) >> (lgw + LGS);
    const int cy = (int)(((float)cell + 0.5f) * A.inv_ex), cx = cell - cy * ex;   // exact: cell < 4096
    const bool ok = cell < A.cells && c < A.E;
    int x = tl.z - halo + cx, y = tl.w - halo + cy;   // the halo wraps, on tiny lattices more than once
    while (x < 0) x += L1;
    while (x >= L1) x -= L1;
    while (y < 0) y += L2;
    while (y >= L2) y -= L2;
    inner[k] = ok && (uint32_t)(cx - halo) < (uint32_t)nx && (uint32_t)(cy - halo) < (uint32_t)ny;
    col[k] = ok ? x : 0;
    const uint32_t site = ok ? (uint32_t)((y * L1 + x) * NSUB + s) : 0u;
    off[k] = (site * NSPIN * (uint32_t)A.Rp + (ok ? (uint32_t)c * NC : 0u)) * 2;
#pragma unroll
    for (int sp = 0; sp < NSPIN; ++sp) {
      v[k][sp] = ld_pack(A.v + Lg.vec_off + off[k] + sp * 2 * A.Rp);
      w[k][sp] = ld_pack(A.w + Lg.vec_off + off[k] + sp * 2 * A.Rp);
    }
    ons[k] = A.onsite ? A.onsite[Lg.site_off + site] : Lg.onsite_const;
    alive[k] = A.mask ? A.mask[Lg.site_off + site] != 0 : true;
  }
  // Peierls factors of the sites' columns (indexed by the A site's cell: a B site's
  // bond class 1 belongs to column x - 1, and the B side takes the conjugate).
  T hre[PHASE ? SPT : 1][3], him[PHASE ? SPT : 1][3];
  if constexpr (PHASE) {
#pragma unroll
    for (int k = 0; k < SPT; ++k)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const int na = (s == 0 || b != 1) ? col[k] : (col[k] == 0 ? L1 - 1 : col[k] - 1);
        const T* ph = A.phase + 2 * (Lg.phase_off + (int64_t)na * 3 + b);
        const T sc = NSPIN == 1 ? C.hop : (T)1;
        hre[k][b] = sc * ph[0];
        him[k][b] = s == 0 ? sc * ph[1] : -sc * ph[1];
      }
  }

  const int cw = NSUB << lgw;                   // items per cell
  const int guard = (ex + 1) * cw;
  const int plane = SPT * kPatchBlock + 2 * guard;   // one spin's packs
  P* cur = reinterpret_cast<P*>(lds) + guard + tid;
  P* nxt = cur + NSPIN * plane;
  // Neighbour offsets: the order of the other step kernels.
  int nb[NNB];
  if constexpr (KIND == KPM_SQUARE) {
    nb[0] = cw;
    nb[1] = -cw;
    nb[2] = ex * cw;
    nb[3] = -ex * cw;
  } else {
    const int o = s == 0 ? ew : -ew;            // to the other sublattice
    nb[0] = o;
    nb[1] = s == 0 ? o - (ex - 1) * cw : o + (ex - 1) * cw;
    nb[2] = s == 0 ? o - ex * cw : o + ex * cw;
  }
#pragma unroll
  for (int k = 0; k < SPT; ++k)
#pragma unroll
    for (int sp = 0; sp < NSPIN; ++sp) cur[sp * plane + k * kPatchBlock] = v[k][sp];
  __syncthreads();

  double acc[HIST ? 1 : KS * 2 * NC];
  if constexpr (!HIST) {
#pragma unroll
    for (int q = 0; q < KS * 2 * NC; ++q) acc[q] = 0.0;
  }
  auto level = [&](int l, T a, T b, bool rw, double* pv, double* pw) {
#pragma unroll
    for (int k = 0; k < SPT; ++k) {
      P vn[NNB][NSPIN], o[NSPIN];
#pragma unroll
      for (int q = 0; q < NNB; ++q)
#pragma unroll
        for (int sp = 0; sp < NSPIN; ++sp) vn[q][sp] = cur[sp * plane + k * kPatchBlock + nb[q]];
      site_step<T, KIND, PHASE, HIST>(a, b, rw, C, hre[PHASE ? k : 0], him[PHASE ? k : 0], ons[k], alive[k], v[k], w[k],
                                      vn, o, inner[k], pv, pw);
#pragma unroll
      for (int sp = 0; sp < NSPIN; ++sp) {
        w[k][sp] = v[k][sp];
        v[k][sp] = o[sp];
        nxt[sp * plane + k * kPatchBlock] = o[sp];
        if constexpr (HIST) {
          if (inner[k]) st_pack(A.out[l] + Lg.vec_off + off[k] + sp * 2 * A.Rp, o[sp]);
        }
      }
    }
    P* t = cur;
    cur = nxt;
    nxt = t;
    lds_barrier();
  };
  if constexpr (HIST) {
#pragma unroll 1
    for (int l = 0; l < A.nlev; ++l) level(l, l == 0 ? A.a1 : (T)2, l == 0 ? A.b1 : (T)1, l > 0 || A.read_w1 != 0, nullptr, nullptr);
  } else {
#pragma unroll
    for (int l = 0; l < KS; ++l) {
      if (l < A.nlev)
        level(l, l == 0 ? A.a1 : (T)2, l == 0 ? A.b1 : (T)1, l > 0 || A.read_w1 != 0, acc + l * 2 * NC,
              acc + l * 2 * NC + NC);
    }
#pragma unroll
    for (int k = 0; k < SPT; ++k)
#pragma unroll
      for (int sp = 0; sp < NSPIN; ++sp) {
        if (inner[k]) {
          st_pack(A.out[1] + Lg.vec_off + off[k] + sp * 2 * A.Rp, v[k][sp]);
          if (A.nlev >= 2) st_pack(A.out[0] + Lg.vec_off + off[k] + sp * 2 * A.Rp, w[k][sp]);
        }
      }
    // The products' sums over the workgroup, per chunk: three exchanges that halve
    // the values a lane holds while they halve the lanes, sums over the remaining
    // lanes of a chunk, then over the waves in order.
    constexpr int NV = KS * 2 * NC;
    static_assert(NV % 8 == 0, "three halvings");
    const int lane = tid & 63;
#pragma unroll
    for (int h = 0; h < 3; ++h) {
      const int bit = 32 >> h, n = NV >> (h + 1);
      const bool up = (lane & bit) != 0;
#pragma unroll
      for (int q = 0; q < n; ++q) {
        const double lo = acc[q], hi = acc[q + n];
        acc[q] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, bit);
      }
    }
    for (int bit = 4; bit >= ew; bit >>= 1)
#pragma unroll
      for (int q = 0; q < NV / 8; ++q) acc[q] += __shfl_xor(acc[q], bit);
    // red[wave][value][chunk]; the guard's barrier above is the level loop's last.
    const int base = ((lane & 32) ? NV / 2 : 0) + ((lane & 16) ? NV / 4 : 0) + ((lane & 8) ? NV / 8 : 0);
    if ((lane & 7) < ew) {
#pragma unroll
      for (int q = 0; q < NV / 8; ++q) lds[(((tid >> 6) * NV + base + q) << lgw) + (lane & 7)] = acc[q];
    }
    __syncthreads();
    // acc order: [level][vv of the NC vectors, then wv].
    for (int i = tid; i < A.nlev * 2 * NC << lgw; i += kPatchBlock) {
      const int cc = i & (ew - 1), val = i >> lgw, l = val / (2 * NC), q = val % (2 * NC);
      double t = 0.0;
#pragma unroll
      for (int wv = 0; wv < kPatchBlock / 64; ++wv) t += lds[((wv * NV + val) << lgw) + cc];
      const int j = q < NC ? 2 * q : 2 * (q - NC) + 1;
      A.part[l * A.part_stride + ((int64_t)A.slot_of[ti] << lgw) * 2 * NC + cc * 2 * NC + j] = t;
    }
  }
}

template <typename T, int KIND, bool PHASE, bool HIST>
static void* pick_patch(int spt) {
  switch (spt) {
    case 1: return (void*)patch_kernel<T, KIND, PHASE, 1, HIST>;
    case 2: return (void*)patch_kernel<T, KIND, PHASE, 2, HIST>;
    default: return (void*)patch_kernel<T, KIND, PHASE, 4, HIST>;

  }
}
template <typename T, bool HIST>
static void* pick_patch_kind(int kind, bool phase, int spt) {
  if (kind == KPM_SQUARE) return pick_patch<T, KPM_SQUARE, false, HIST>(spt);
  if (kind == KPM_HONEYCOMB)
    return phase ? pick_patch<T, KPM_HONEYCOMB, true, HIST>(spt) : pick_patch<T, KPM_HONEYCOMB, false, HIST>(spt);
  return phase ? pick_patch<T, KPM_HONEYCOMB_SPIN, true, HIST>(spt)
               : pick_patch<T, KPM_HONEYCOMB_SPIN, false, HIST>(spt);
}

}  // namespace kpm
