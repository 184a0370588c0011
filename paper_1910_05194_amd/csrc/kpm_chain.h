// Site arithmetic of the conductivity chains, shared by the row sweeps (kpm_chain.hip)
// and the patches (kpm_patch_chain.hip).
#pragma once

#include "kpm_stencil.h"

namespace kpm {

// Hopping coefficients of one thread's orbital (per tile): the complex
// coefficient of the value of neighbour k, spin s2, in the result for the
// thread's spin, Peierls phase and hopping folded in.  Spinless: hop *
// exp(i theta_k).  Spinful: exp(i theta_k) times the 2 x 2 Rashba block
// entry, B_k[sp][s2] on sublattice A and conj(B_k[s2][sp]) on sublattice B.
template <typename T, int KIND>
struct Coef {
  static constexpr int NNB = KindTraits<KIND>::NNB, NSPIN = KindTraits<KIND>::NSPIN;
  T re[NNB][NSPIN], im[NNB][NSPIN];
  T vc[NNB];   // velocity weights (mode 1)
};

// One orbital: out = a (H~ v) - b w and, in mode 1, the velocity stencil of
// v, vout = vel_scale sum_k d_k term_k, where term_k is the hop from
// neighbour k (both spins) applied to its values.
template <typename T, int KIND, int MODE>
__device__ inline void chain_site(T a, T b, bool read_w, const Coef<T, KIND>& C, T ons, T vel_scale, bool alive,
                                  const Pack<T>& vo, const Pack<T>& wo,
                                  const Pack<T> (&vn)[KindTraits<KIND>::NNB][KindTraits<KIND>::NSPIN], Pack<T>& out,
                                  Pack<T>& vout) {
  constexpr int NC = Pack<T>::NC;
  constexpr int NSPIN = KindTraits<KIND>::NSPIN;
  constexpr int NNB = KindTraits<KIND>::NNB;
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    T hr = ons * vo.v[2 * j], hi = ons * vo.v[2 * j + 1];
    T gr = 0, gi = 0;
    // Complex products as chains of FMAs (the compiler may not reassociate
    // a sum of products into them): four per coefficient and value.  Mode 0
    // adds every term straight into the result; mode 1 keeps each
    // neighbour's term for the velocity sum.
#pragma unroll
    for (int k = 0; k < NNB; ++k) {
      if constexpr (MODE == 1) {
        T tr = C.re[k][0] * vn[k][0].v[2 * j];
        T ti = C.re[k][0] * vn[k][0].v[2 * j + 1];
        tr = fma(-C.im[k][0], vn[k][0].v[2 * j + 1], tr);
        ti = fma(C.im[k][0], vn[k][0].v[2 * j], ti);
#pragma unroll
        for (int s2 = 1; s2 < NSPIN; ++s2) {
          tr = fma(C.re[k][s2], vn[k][s2].v[2 * j], tr);
          tr = fma(-C.im[k][s2], vn[k][s2].v[2 * j + 1], tr);
          ti = fma(C.re[k][s2], vn[k][s2].v[2 * j + 1], ti);
          ti = fma(C.im[k][s2], vn[k][s2].v[2 * j], ti);
        }
        hr += tr;
        hi += ti;
        gr = fma(C.vc[k], tr, gr);
        gi = fma(C.vc[k], ti, gi);
      } else {
#pragma unroll
        for (int s2 = 0; s2 < NSPIN; ++s2) {
          hr = fma(C.re[k][s2], vn[k][s2].v[2 * j], hr);
          hr = fma(-C.im[k][s2], vn[k][s2].v[2 * j + 1], hr);
          hi = fma(C.re[k][s2], vn[k][s2].v[2 * j + 1], hi);
          hi = fma(C.im[k][s2], vn[k][s2].v[2 * j], hi);
        }
      }
    }
    T orr = a * hr, oi = a * hi;
    if (read_w) {
      orr -= b * wo.v[2 * j];
      oi -= b * wo.v[2 * j + 1];
    }
    if (!alive) {
      orr = 0;
      oi = 0;
      gr = 0;
      gi = 0;
    }
    out.v[2 * j] = orr;
    out.v[2 * j + 1] = oi;
    if constexpr (MODE == 1) {
      vout.v[2 * j] = vel_scale * gr;
      vout.v[2 * j + 1] = vel_scale * gi;
    }
  }
}

}  // namespace kpm
