// Moment-extrapolation MLP: n_in -> n_hid -> n_hid -> n_out with exact GELU,
// trained and evaluated on the GPU by the kernels below.  It maps the first
// n_in Chebyshev moments of a DOS to the next n_out moments, so that fewer
// recursion steps are needed; the full recursion remains the reference and
// the fallback.  (The paper has no learned component.)
//
// Kernels: an FP32 MFMA GEMM (v_mfma_f32_16x16x4_f32) with the standardisation
// of the inputs folded into its loads and bias, GELU, loss, GELU backward or
// the Adam update into its epilogue (training and FP32 inference); a BF16 MFMA GEMM with FP32
// accumulation (v_mfma_f32_32x32x16_bf16) that stages a weight panel in LDS
// (inference).  Every reduction runs in a fixed order (bitwise reproducible).

#include "kpm_internal.h"
#include "kpm_stencil.h"

#include <cmath>
#include <cstring>
#include <new>
#include <vector>

namespace kpm {

typedef float f32x4m __attribute__((ext_vector_type(4)));
typedef float f32x16m __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8m __attribute__((ext_vector_type(8)));

constexpr int kGemmThreads = 256;  // four waves
constexpr int kChunk = 64;         // contraction indices per LDS stage (32 in the products of large batches)
constexpr int kLossBlocks = 256;   // partial sums of the stand-alone loss
constexpr double kBeta1 = 0.9, kBeta2 = 0.999;

enum { EPI_BIAS = 0, EPI_GELU = 1, EPI_LOSS = 2, EPI_GELU_BACK = 3, EPI_GRAD = 4, EPI_ADAM = 5 };

__device__ inline float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ inline float gelu_grad_f(float x) {
  const float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
  const float pdf = 0.39894228040143268f * expf(-0.5f * x * x);
  return cdf + x * pdf;
}

struct AdamArgs {
  float lr = 0.f, c1 = 1.f, c2 = 1.f;   // step size, bias corrections 1/(1 - beta^t)
};

// One product C[M][N] = op(A) op(B) with its epilogue's operands.
struct Gemm {
  const float* A = nullptr;   // op(A) = A [M][K], or A^T with A stored [K][M]
  const float* B = nullptr;   // op(B) = B [K][N], or B^T with B stored [N][K]
  int lda = 0, ldb = 0, M = 0, N = 0, K = 0;
  int tm = 0, tn = 0;         // output tiles
  const float *x_shift = nullptr, *x_scale = nullptr;   // A holds inputs to be standardised by feature (or null)
  float* C = nullptr;         // EPI_BIAS, EPI_GELU, EPI_LOSS (the loss gradient), EPI_GELU_BACK, EPI_GRAD
  int ldc = 0;
  float* Z = nullptr;         // pre-activation: written by EPI_GELU, read by EPI_GELU_BACK
  const float* bias = nullptr;
  const float *y_shift = nullptr, *y_scale = nullptr;   // EPI_BIAS: output units; EPI_LOSS: target standardisation
  const float *T = nullptr, *w = nullptr;               // EPI_LOSS
  double* partial = nullptr;
  float* bias_grad = nullptr;                           // EPI_GRAD: column sums of op(B)
  float *par = nullptr, *m = nullptr, *v = nullptr;     // EPI_ADAM: the weights
  float *bpar = nullptr, *bm = nullptr, *bv = nullptr;  //           and the biases
  AdamArgs ad;
};

// Adam (Kingma & Ba 2015).  The FMAs are written out: a training run is the same
// to the bit wherever the compiler puts this.
__device__ inline void adam_update(float g, const AdamArgs& a, float* p, float* m, float* v) {
  const float b1 = (float)kBeta1, b2 = (float)kBeta2;
  const float mi = fmaf(1.f - b1, g, b1 * *m);
  const float vi = fmaf(g, (1.f - b2) * g, b2 * *v);
  *m = mi;
  *v = vi;
  *p -= a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + 1e-8f);
}

// LDS of one product: two stages of the operand panels, k-major.
// (80 floats a row are two workgroups per CU at CH = 64; 81 would be one.)
template <int CH>
struct GemmLds {
  static constexpr int kRow = CH == kChunk ? 80 : 81;
  float a[2][CH * kRow], b[2][CH * kRow];
};

// Staging of a panel op(X)[k0 .. k0 + CH - 1][x0 .. x0 + W - 1] by 256 threads,
// CH W / 1024 groups of four values each: KC = the operand's rows are contiguous in k
// (CH / 4 threads take the k of one index), else contiguous in the index (W / 4
// threads take the indices of one k).  Values outside are zero.
// LDS pitch: an MFMA operand read takes 16 indices of four k rows, the transposed
// (KC) store 16 k quads of four indices.  W + 16 puts the four rows of a read in
// different quarters of the 64 banks; the store of a KC panel also needs an odd
// pitch (all 64 banks, and reads with at most one bank shared by two rows).
// Loads go through buffer resources: an element outside gets an offset past the
// range, which reads as zero, so that no branch (whose merge would wait for every
// load in flight) stands around a load.  NORM: the values are standardised by
// feature on their way to LDS; the features run along k (KC) or the index.
template <bool KC, bool VEC, int W, bool NORM, int CH>
struct Panel {
  static constexpr int G = CH * W / 1024, kQuads = CH / 4;
  static constexpr int kPitch = W + 16 + (KC ? 1 : 0);
  float x[G][4], sh[NORM ? G : 1][4], sc[NORM ? G : 1][4];
  __device__ static int idx(int g) { return KC ? (int)(threadIdx.x / kQuads) + (256 / kQuads) * g : 4 * (int)(threadIdx.x % (W / 4)); }
  __device__ static int kk(int g) {
    return KC ? 4 * (int)(threadIdx.x % kQuads) : (int)(threadIdx.x / (W / 4)) + (1024 / W) * g;
  }
  __device__ static void load4(__amdgpu_buffer_rsrc_t r, uint32_t off, float (&v)[4]) {
    const float4 u = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
    v[0] = u.x; v[1] = u.y; v[2] = u.z; v[3] = u.w;
  }
  __device__ void load(const Gemm& gm, const float* __restrict__ P, int ld, int x0, int nx, int k0, int nk) {
    const __amdgpu_buffer_rsrc_t r = row_rsrc(KC ? P + (int64_t)x0 * ld + k0 : P + (int64_t)k0 * ld + x0, 0x7fffffffu);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int i = idx(g), k = kk(g);
      const uint32_t off = 4u * (KC ? (uint32_t)i * ld + k : (uint32_t)k * ld + i);
      if constexpr (VEC) {
        load4(r, ((x0 + i < nx) & (k0 + k < nk)) ? off : kOOB, x[g]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          x[g][e] = buf_ld_scalar<float>(
              r, (((KC ? x0 + i : x0 + i + e) < nx) & ((KC ? k0 + k + e : k0 + k) < nk)) ? off + 4u * e : kOOB);
      }
      if constexpr (NORM) {
        const int f0 = KC ? k0 : x0;
        const uint32_t bytes = 4u * (uint32_t)((KC ? nk : nx) - f0);
        load4(row_rsrc(gm.x_shift + f0, bytes), 4u * (KC ? k : i), sh[g]);
        load4(row_rsrc(gm.x_scale + f0, bytes), 4u * (KC ? k : i), sc[g]);
      }
    }
  }
  __device__ void standardise(int x0, int nx, int k0, int nk) {
    if constexpr (NORM) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = x0 + idx(g) + (KC ? 0 : e) < nx && k0 + kk(g) + (KC ? e : 0) < nk;
          x[g][e] = in ? (x[g][e] - sh[g][e]) / sc[g][e] : 0.f;
        }
    }
  }
  __device__ void store(float* dst) const {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if constexpr (KC) {
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[(kk(g) + e) * kPitch + idx(g)] = x[g][e];
      } else {
        *reinterpret_cast<float4*>(&dst[kk(g) * kPitch + idx(g)]) = make_float4(x[g][0], x[g][1], x[g][2], x[g][3]);
      }
    }
  }
};

// One output tile of 32 NW x 32 NW by the four waves of a workgroup (2 x 2, each
// NW x NW MFMA tiles of 16 x 16), contraction indices in ascending order into
// one accumulator per output (the order fixes the result to the bit).  Panels
// of 64 indices go global memory -> registers (two panels ahead) -> one of two
// LDS stages, one barrier per panel.
//
// At the training sizes (batch 256, widths 256..1792) a product is 0.1..0.9
// GFLOP, 1..6 us of MFMA time over the whole chip, and its accumulation chain
// (up to 1792 indices) is serial: 16x16x4 tiles take 8 clocks per index of
// that chain where 32x32x2 tiles take 32, and 32 x 32 outputs per workgroup
// give 256..448 workgroups where 64 x 64 gave 64..112.  Those, with one stage
// of 32 indices between two barriers and no loads in flight, took 38..214 us a
// product; these take 9..21 us, 30 % of it MFMA (the rest: LDS and L2 latency at
// one wave per SIMD), and the weight updates 29..36 us (half of it Adam's 24 bytes
// per parameter).  24 training steps: 28.1 -> 3.8 ms.
template <bool TA, bool TB, int NW, int EPI, bool VEC, bool NORM, int CH = kChunk>
__device__ inline void gemm_tile(const Gemm& g, int tile, GemmLds<CH>& lds) {
  constexpr int W = 32 * NW;
  const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
  const int wave = threadIdx.x >> 6;
  const int wi = (wave & 1) * 16 * NW, wj = (wave >> 1) * 16 * NW;
  const int m0 = (tile % g.tm) * W, n0 = (tile / g.tm) * W;
  const int chunks = (g.K + CH - 1) / CH;
  using PA = Panel<!TA, VEC, W, NORM, CH>;
  using PB = Panel<TB, VEC, W, false, CH>;
  static_assert(PA::kPitch <= GemmLds<CH>::kRow && PB::kPitch <= GemmLds<CH>::kRow, "panels fit their stages");
  PA pa[2];
  PB pb[2];
  auto load = [&](int c, PA& a, PB& b) {
    a.load(g, g.A, g.lda, m0, g.M, c * CH, g.K);
    b.load(g, g.B, g.ldb, n0, g.N, c * CH, g.K);
  };
  auto store = [&](int c, PA& a, const PB& b, int st) {
    a.standardise(m0, g.M, c * CH, g.K);
    a.store(lds.a[st]);
    b.store(lds.b[st]);
  };
  f32x4m acc[NW][NW];
#pragma unroll
  for (int i = 0; i < NW; ++i)
#pragma unroll
    for (int j = 0; j < NW; ++j) acc[i][j] = f32x4m{};
  // Column sums of op(B) (bias gradients), in ascending order too.
  const bool colsum = (EPI == EPI_GRAD || EPI == EPI_ADAM) && m0 == 0 && (int)threadIdx.x < W;
  float col = 0.f;
  auto product = [&](int st) {
    // Operands of CH / 8 steps of four indices at a time, the next batch on its way
    // from LDS while one is multiplied (with one wave per SIMD a read before each
    // MFMA costs its whole latency).
    constexpr int H = CH / 8;
    float a[2][H][NW], b[2][H][NW];
    auto read = [&](int h, int set) {
#pragma unroll
      for (int s = 0; s < H; ++s)
#pragma unroll
        for (int i = 0; i < NW; ++i) {
          a[set][s][i] = lds.a[st][(4 * (H * h + s) + q) * PA::kPitch + wi + 16 * i + r];
          b[set][s][i] = lds.b[st][(4 * (H * h + s) + q) * PB::kPitch + wj + 16 * i + r];
        }
    };
    read(0, 0);
#pragma unroll
    for (int h = 0; h < CH / (4 * H); ++h) {
      if (h + 1 < CH / (4 * H)) read(h + 1, (h + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < H; ++s)
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
          for (int j = 0; j < NW; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h & 1][s][i], b[h & 1][s][j], acc[i][j], 0, 0, 0);
    }
    if (colsum) {
#pragma unroll 16
      for (int k = 0; k < CH; ++k) col += lds.b[st][k * PB::kPitch + threadIdx.x];
    }
  };
  load(0, pa[0], pb[0]);
  if (1 < chunks) load(1, pa[1], pb[1]);
  store(0, pa[0], pb[0], 0);
  if (2 < chunks) load(2, pa[0], pb[0]);
  // Element e of a tile: row 4 q + e, column r.  What the epilogue reads is loaded
  // now, so that it arrives under the main loop (after the loop the loads would also
  // have to wait, one element after another, for the stores they may alias).
  constexpr int NE = 4 * NW * NW;
  constexpr bool kBias = EPI == EPI_BIAS || EPI == EPI_GELU || EPI == EPI_LOSS;
  constexpr bool kScale = EPI == EPI_BIAS || EPI == EPI_LOSS;
  int64_t o[NE];
  bool in[NE];
  float e0[NE], e1[NE], e2[NE];   // LOSS: T, w;  GELU_BACK: Z;  ADAM: p, m, v
  float bias[NW], ys[NW], yc[NW];
#pragma unroll
  for (int tj = 0; tj < NW; ++tj) {
    const int j = min(n0 + wj + 16 * tj + r, g.N - 1);
    bias[tj] = kBias ? g.bias[j] : 0.f;
    ys[tj] = (kScale && g.y_shift) ? g.y_shift[j] : 0.f;
    yc[tj] = (kScale && g.y_shift) ? g.y_scale[j] : 1.f;
  }
#pragma unroll
  for (int x = 0; x < NE; ++x) {
    const int e = x & 3, ti = (x >> 2) / NW, tj = (x >> 2) % NW;
    const int i = m0 + wi + 16 * ti + 4 * q + e, j = n0 + wj + 16 * tj + r;
    in[x] = (i < g.M) & (j < g.N);
    o[x] = (int64_t)i * g.ldc + j;
    const int64_t oc = in[x] ? o[x] : 0;
    if constexpr (EPI == EPI_LOSS) {
      e0[x] = g.T[oc];
      e1[x] = g.w[min(j, g.N - 1)];
    }
    if constexpr (EPI == EPI_GELU_BACK) e0[x] = g.Z[oc];
    if constexpr (EPI == EPI_ADAM) {
      e0[x] = g.par[oc];
      e1[x] = g.m[oc];
      e2[x] = g.v[oc];
    }
  }
  // Chunk c is in LDS stage c % 2, chunks c + 1 and c + 2 are on their way.
  auto step = [&](int c, PA& a, PB& b, int st) {
    lds_barrier();
    if (c + 1 < chunks) store(c + 1, a, b, st ^ 1);
    if (c + 3 < chunks) load(c + 3, a, b);
    product(st);
  };
  int c = 0;
  for (; c + 2 <= chunks; c += 2) {
    step(c, pa[1], pb[1], 0);
    step(c + 1, pa[0], pb[0], 1);
  }
  if (c < chunks) step(c, pa[1], pb[1], 0);
  double loss = 0.0;
#pragma unroll
  for (int x = 0; x < NE; ++x) {
    const int ti = (x >> 2) / NW, tj = (x >> 2) % NW;
    if (!in[x]) continue;
    float y = acc[ti][tj][x & 3];
    if constexpr (EPI == EPI_BIAS) {
      y += bias[tj];
      if (g.y_shift) y = ys[tj] + yc[tj] * y;
      g.C[o[x]] = y;
    } else if constexpr (EPI == EPI_GELU) {
      y += bias[tj];
      g.Z[o[x]] = y;
      g.C[o[x]] = gelu_f(y);
    } else if constexpr (EPI == EPI_LOSS) {
      // Loss and its gradient 2 w_j^2 (Y - T) / (B n_out).  With standardisation the
      // network predicts (y - my)/sy and (w (y - t))^2 = (w sy (y' - t'))^2.
      y += bias[tj];
      float t = e0[x], w = e1[x];
      if (g.y_shift) {
        t = (t - ys[tj]) / yc[tj];
        w *= yc[tj];
      }
      const float d = y - t;
      g.C[o[x]] = (float)(2.0 / ((double)g.M * g.N)) * w * w * d;
      const double er = (double)w * (double)d;
      loss += er * er;
    } else if constexpr (EPI == EPI_GELU_BACK) {
      g.C[o[x]] = y * gelu_grad_f(e0[x]);
    } else if constexpr (EPI == EPI_GRAD) {
      g.C[o[x]] = y;
    } else {
      adam_update(y, g.ad, &e0[x], &e1[x], &e2[x]);
      g.par[o[x]] = e0[x];
      g.m[o[x]] = e1[x];
      g.v[o[x]] = e2[x];
    }
  }
  if (colsum && n0 + (int)threadIdx.x < g.N) {
    const int j = n0 + threadIdx.x;
    if constexpr (EPI == EPI_GRAD) g.bias_grad[j] = col;
    if constexpr (EPI == EPI_ADAM) adam_update(col, g.ad, g.bpar + j, g.bm + j, g.bv + j);
  }
  if constexpr (EPI == EPI_LOSS) {
    __syncthreads();
    double* red = reinterpret_cast<double*>(&lds);
    red[threadIdx.x] = loss;
    __syncthreads();
    for (int s = kGemmThreads / 2; s > 0; s >>= 1) {
      if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0) g.partial[tile] = red[0] / ((double)g.M * g.N);
  }
}

// Workgroup b runs on XCD b % 8: each XCD takes a contiguous range of tiles
// (rows fastest), so that the tiles sharing a panel of the larger operand, the
// weights, read it through one L2.
__device__ inline int xcd_tile() { return (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)); }

template <bool TA, bool TB, int NW, int EPI, bool VEC, bool NORM, int CH = kChunk>
__global__ void __launch_bounds__(kGemmThreads) mlp_gemm(Gemm g) {
  __shared__ GemmLds<CH> lds;
  const int tile = xcd_tile();
  if (tile < g.tm * g.tn) gemm_tile<TA, TB, NW, EPI, VEC, NORM, CH>(g, tile, lds);
}

__device__ inline void sum_partials(const double* partial, int n, double* out, double* red) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += partial[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = red[0];
}

// Two independent products in one launch: the activation gradient
// dZ = (dY W^T) gelu'(Z) of a layer and the weight gradient (or Adam update) of
// the layer above it, whose weights the first no longer needs.
template <int EPIW, bool VEC>
__global__ void __launch_bounds__(kGemmThreads) mlp_back_pair(Gemm act, Gemm wgt) {
  __shared__ GemmLds<kChunk> lds;
  const int tile = xcd_tile(), na = act.tm * act.tn;
  if (tile < na) gemm_tile<false, true, 1, EPI_GELU_BACK, VEC, false>(act, tile, lds);
  else if (tile - na < wgt.tm * wgt.tn) gemm_tile<true, false, 2, EPIW, VEC, false>(wgt, tile - na, lds);
}

// The weight gradients (or updates) of two layers, and the sum of the loss
// partials by one more workgroup.
template <int EPIW, bool VEC, bool NORM>
__global__ void __launch_bounds__(kGemmThreads) mlp_weight_pair(Gemm g1, Gemm g2, const double* partial, int n_partial,
                                                                double* loss) {
  __shared__ GemmLds<kChunk> lds;
  const int tile = xcd_tile(), n1 = g1.tm * g1.tn, n2 = g2.tm * g2.tn;
  if (tile < n1) gemm_tile<true, false, 2, EPIW, VEC, false>(g1, tile, lds);
  else if (tile - n1 < n2) gemm_tile<true, false, 2, EPIW, VEC, NORM>(g2, tile - n1, lds);
  else if (tile == n1 + n2) sum_partials(partial, n_partial, loss, reinterpret_cast<double*>(&lds));
}

// ---------------------------------------------------------------------------
// BF16 inference: out = act(A W + b) with A and W rounded to BF16, FP32
// accumulation over k in ascending blocks of 16 in one accumulator per output
// (the order fixes the result, and with it the rounding of the next layer's
// operands).  One workgroup owns 32 columns: its 512 threads load the FP32
// weight panel [<= 1024][32], all of it in flight at once, and lay it down in
// LDS as BF16 in MFMA operand order; each wave then runs 32 rows (8 x 32 rows
// per workgroup; batches beyond that take more workgroups).  Hidden
// activations are stored as the BF16 values the next layer uses, rows padded
// to whole 32-column tiles with zeros.
//
// Bound: reading 12.6 MB of weights once (3 us at HBM rate) from 32..56
// workgroups, i.e. by how many loads a workgroup keeps in flight.  With 32
// indices per stage and two barriers a stage (64 x 64 tiles) a layer of 1024
// took 75..115 us at batch 64, now 11..12 us (the first layer 17, half of it the
// divisions of the standardisation).
// ---------------------------------------------------------------------------
constexpr int kPanelK = 1024;   // weight rows per LDS panel (64 KiB)
constexpr int kInferThreads = 512;

// KIND 0: A is FP32 (inputs, standardised when x_shift is given), 1: the same with
// 16-byte aligned rows, 2: A is BF16, rows padded with zeros to lda.
// A row's values k .. k + 7 (k < K; past K zero) through a buffer resource at the
// wave's first row (32-bit offsets: 64-bit addresses of the loads in flight would
// take more registers than the data).
template <int KIND>
struct InferOperand {
  float x[8];
  __device__ void load(__amdgpu_buffer_rsrc_t r, uint32_t row_off, int k, int K) {
    if constexpr (KIND == 1) {
#pragma unroll
      for (int e = 0; e < 8; e += 4) {
        const float4 u = __builtin_bit_cast(
            float4, __builtin_amdgcn_raw_buffer_load_b128(r, k + e < K ? row_off + 4u * (k + e) : kOOB, 0, 0));
        x[e] = u.x; x[e + 1] = u.y; x[e + 2] = u.z; x[e + 3] = u.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = buf_ld_scalar<float>(r, k + e < K ? row_off + 4u * (k + e) : kOOB);
    }
  }
  // norm: (shift, scale) of the features from this operand's first on, or null.
  __device__ bf16x8m value(const float2* norm) const {
    bf16x8m a;
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = norm ? (__bf16)((x[e] - norm[e].x) / norm[e].y) : (__bf16)x[e];
    return a;
  }
};
template <>
struct InferOperand<2> {
  bf16x8m x;
  __device__ void load(__amdgpu_buffer_rsrc_t r, uint32_t row_off, int k, int K) {
    x = __builtin_bit_cast(bf16x8m, __builtin_amdgcn_raw_buffer_load_b128(r, k < K ? row_off + 2u * k : kOOB, 0, 0));
  }
  __device__ bf16x8m value(const float2*) const { return x; }
};

template <int KIND, bool HIDDEN>
__global__ void __launch_bounds__(kInferThreads) mlp_infer_kernel(const void* A, int lda, const float* __restrict__ W,
                                                                  int ldw, const float* __restrict__ bias, int M, int N,
                                                                  int K, const float* x_shift, const float* x_scale,
                                                                  const float* y_shift, const float* y_scale, void* out,
                                                                  int ldo) {
  __shared__ bf16x8m panel[kPanelK / 8][32];
  __shared__ float2 norm[KIND == 2 ? 1 : kPanelK];
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n0 = blockIdx.x * 32, m0 = blockIdx.y * 256 + wave * 32;
  const int pj = threadIdx.x & 31, po = threadIdx.x >> 5;   // panel column and octet of this thread
  const bool active = m0 < M;
  f32x16m acc = f32x16m{};
  for (int k0 = 0; k0 < K; k0 += kPanelK) {
    const int kc = min(kPanelK, K - k0);
    const int steps = (kc + 63) / 64 * 4;   // of 16, in whole groups of four; operands past kc are zero
    if (k0 > 0) __syncthreads();
    // The first operand rows and the whole weight panel, in flight together.
    constexpr int D = KIND == 2 ? 16 : 8;   // steps of 16 whose operands are in flight
    constexpr int Q = 4;                    // steps whose LDS operands are read ahead
    constexpr int kSize = KIND == 2 ? 2 : 4;
    const __amdgpu_buffer_rsrc_t ra =
        row_rsrc(reinterpret_cast<const char*>(A) + ((int64_t)min(m0, M - 1) * lda + k0) * kSize, 0x7fffffffu);
    const uint32_t row_off = (uint32_t)max(min(r, M - 1 - m0), 0) * lda * kSize;
    InferOperand<KIND> a[D];
    auto load_a = [&](int s0, auto lo, auto hi) {
#pragma unroll
      for (int d = lo(); d < hi(); ++d) a[d].load(ra, row_off, 16 * (s0 + d) + 8 * h, kc);
    };
    float x[kPanelK / 128][8];
    const __amdgpu_buffer_rsrc_t rw = row_rsrc(W + (int64_t)k0 * ldw + n0, 0x7fffffffu);
    if (kc % 128 == 0 && n0 + 32 <= N) {
      const uint32_t off = 4u * ((uint32_t)(8 * po) * ldw + pj);
#pragma unroll
      for (int q = 0; q < kPanelK / 128; ++q)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (128 * q < kc)
            x[q][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw, off, 4 * (128 * q + e) * ldw, 0));
          else
            x[q][e] = 0.f;
    } else {
#pragma unroll
      for (int q = 0; q < kPanelK / 128; ++q) {
        int kq = 8 * (po + 16 * q);
        asm volatile("" : "+v"(kq));   // (not hoisted out of the panel loop: 64 offsets would spill)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          x[q][e] = buf_ld_scalar<float>(rw, (kq + e < kc) & (n0 + pj < N) ? 4u * ((uint32_t)(kq + e) * ldw + pj) : kOOB);
      }
    }
    std::integral_constant<int, 0> d0;
    std::integral_constant<int, D / 2> d1;
    std::integral_constant<int, D> d2;
    if (active) load_a(0, d0, d1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (KIND != 2) {
      if (x_shift)
        for (int k = threadIdx.x; k < 16 * steps; k += kInferThreads)
          norm[k] = k < kc ? make_float2(x_shift[k0 + k], x_scale[k0 + k]) : make_float2(0.f, 1.f);
    }
#pragma unroll
    for (int q = 0; q < kPanelK / 128; ++q) {
      const int o = po + 16 * q;
      bf16x8m b;
#pragma unroll
      for (int e = 0; e < 8; ++e) b[e] = (__bf16)x[q][e];
      if (o < 2 * steps) panel[o][pj] = b;
    }
    if (active) load_a(0, d1, d2);   // (in the panel values' registers)
    __syncthreads();
    if (active) {
      for (int s0 = 0; s0 < steps; s0 += D) {
        if (s0 > 0) load_a(s0, d0, d2);
        bf16x8m b[2][Q];
        auto read_b = [&](int s, bf16x8m (&dst)[Q]) {
#pragma unroll
          for (int d = 0; d < Q; ++d) dst[d] = panel[2 * (s + d) + h][r];
        };
        read_b(s0, b[0]);
#pragma unroll
        for (int g = 0; g < D; g += Q) {
          if (s0 + g >= steps) break;
          if (g + Q < D && s0 + g + Q < steps) read_b(s0 + g + Q, b[(g / Q + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int d = 0; d < Q; ++d)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                a[g + d].value(x_shift ? &norm[KIND == 2 ? 0 : 16 * (s0 + g + d) + 8 * h] : nullptr), b[(g / Q) & 1][d],
                acc, 0, 0, 0);
        }
      }
    }
  }
  if (!active) return;
  const int j = n0 + r;
  const float bj = j < N ? bias[j] : 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int i = m0 + 8 * (e >> 2) + 4 * h + (e & 3);
    if (i >= M) continue;
    float v = acc[e] + bj;
    if constexpr (HIDDEN) {
      reinterpret_cast<__bf16*>(out)[(int64_t)i * ldo + j] = j < N ? (__bf16)gelu_f(v) : (__bf16)0.f;
    } else if (j < N) {
      if (y_shift) v = y_shift[j] + y_scale[j] * v;
      reinterpret_cast<float*>(out)[(int64_t)i * ldo + j] = v;
    }
  }
}

// Per-block partial sums (FP64) of the loss 1/(B n_out) sum (w_j (Y - T))^2.
__global__ void mlp_loss_kernel(const float* Y, const float* T, const float* w, int Bn, int n_out, double* partial) {
  __shared__ double red[256];
  const int64_t n = (int64_t)Bn * n_out;
  const double inv = 1.0 / (double)n;
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float d = Y[i] - T[i];
    const double e = (double)w[(int)(i % n_out)] * (double)d;
    acc += e * e;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0] * inv;
}

// err[b] = sqrt(sum_j (w_j (Y_bj - R_bj))^2) / sqrt(sum_j (w_j R_bj)^2) over the
// first n_cmp of the n_out columns of Y, or with noise given,
// sqrt(sum_j (w_j (Y_bj - R_bj))^2) / (noise_b sqrt(sum_j w_j^2)); one
// workgroup per row, FP64 sums in a fixed-order tree.
__global__ void rel_error_kernel(const float* Y, int n_out, const double* R, int n_cmp, const float* w,
                                 const double* noise, double* err) {
  __shared__ double num[256], den[256];
  const int b = blockIdx.x;
  double a = 0.0, d = 0.0;
  for (int j = threadIdx.x; j < n_cmp; j += blockDim.x) {
    const double r = R[(int64_t)b * n_cmp + j], wj = w[j];
    const double e = wj * ((double)Y[(int64_t)b * n_out + j] - r);
    a += e * e;
    d += noise ? wj * wj : (wj * r) * (wj * r);
  }
  num[threadIdx.x] = a;
  den[threadIdx.x] = d;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      num[threadIdx.x] += num[threadIdx.x + st];
      den[threadIdx.x] += den[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) err[b] = sqrt(num[0]) / fmax((noise ? noise[b] : 1.0) * sqrt(den[0]), 1e-300);
}

// out = the sum of n partials: 256 strided sums, then a fixed-order tree.
__global__ void sum_partials_kernel(const double* partial, int n, double* out) {
  __shared__ double red[256];
  sum_partials(partial, n, out, red);
}

// He-uniform initialisation from the SplitMix64 stream (purpose 5): W ~ U(-s, s), s = sqrt(3/fan_in).
__global__ void init_uniform_kernel(float* p, int64_t n, uint64_t key, float scale) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  p[i] = (float)((2.0 * sm_uniform(key, (uint64_t)i) - 1.0) * scale);
}

// Column statistics of a [n][cols] table (FP64, fixed order): shift = mean,
// scale = standard deviation (1 where it vanishes).  A workgroup takes 16
// columns and splits the rows over 64 threads each (one thread per column left
// the chip idle: 2.5 ms at 6144 x 1792).
constexpr int kStatCols = 16;
__global__ void __launch_bounds__(1024) column_stats_kernel(const float* X, int64_t n, int cols, float* shift,
                                                            float* scale) {
  __shared__ double red[64][kStatCols];
  const int c = threadIdx.x % kStatCols, q = threadIdx.x / kStatCols;
  const int j = blockIdx.x * kStatCols + c;
  const bool in = j < cols;
  auto total = [&](double x) {
    __syncthreads();
    red[q][c] = x;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < 64; ++i) s += red[i][c];
    return s;
  };
  double s = 0.0;
  if (in)
    for (int64_t i = q; i < n; i += 64) s += X[i * cols + j];
  const double mean = total(s) / (double)n;
  double v = 0.0;
  if (in)
    for (int64_t i = q; i < n; i += 64) {
      const double d = X[i * cols + j] - mean;
      v += d * d;
    }
  const double sd = sqrt(total(v) / (double)n);
  if (in && q == 0) {
    shift[j] = (float)mean;
    scale[j] = sd > 0.0 ? (float)sd : 1.0f;
  }
}

__global__ void fill_f32(float* p, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace kpm

struct kpm_mlp {
  int n_in = 0, n_hid = 0, n_out = 0;
  int64_t off[6] = {0, 0, 0, 0, 0, 0};   // W1 b1 W2 b2 W3 b3 offsets (floats)
  int64_t n_par = 0;
  float* par = nullptr;
  float* grad = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  int64_t t = 0;
  int cap_b = 0;                          // workspace capacity (batch rows)
  float *Z1 = nullptr, *A1 = nullptr, *Z2 = nullptr, *A2 = nullptr, *Y = nullptr, *dY = nullptr;
  float *dZ1 = nullptr, *dZ2 = nullptr;
  double* partial = nullptr;              // loss partials (one per workgroup of the kernel that forms them)
  double* loss_dev = nullptr;
  // Optional per-column standardisation of inputs and outputs.
  bool scaled = false;
  float *x_shift = nullptr, *x_scale = nullptr, *y_shift = nullptr, *y_scale = nullptr;
};

namespace kpm {

static int mlp_reserve(kpm_mlp* N, int B) {
  if (B <= N->cap_b) return KPM_OK;
  // Drop the old workspace first: after a failed allocation the network holds
  // no workspace (cap_b = 0), and the next call allocates it again.
  N->cap_b = 0;
  float** bufs[] = {&N->Z1, &N->A1, &N->Z2, &N->A2, &N->Y, &N->dY, &N->dZ1, &N->dZ2};
  for (float** b : bufs) {
    (void)::kpm::dev_free(*b);
    *b = nullptr;
  }
  (void)::kpm::dev_free(N->partial);
  N->partial = nullptr;
  // A1 and A2 also hold the BF16 activations of the inference kernels, rows
  // padded to whole 32-column tiles (at least 16 floats a row).
  const int64_t h = (int64_t)B * N->n_hid, o = (int64_t)B * N->n_out, a = (int64_t)B * std::max(N->n_hid, 16);
  const int64_t n_part = std::max<int64_t>(kLossBlocks, ceil_div(B, 32) * ceil_div(N->n_out, 32));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->Z1, h * 4, false));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->A1, a * 4, false));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->Z2, h * 4, false));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->A2, a * 4, false));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->Y, o * 4, false));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->dY, o * 4, false));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->dZ1, h * 4, false));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->dZ2, h * 4, false));
  KPM_TRY_HIP(::kpm::dev_malloc(&N->partial, n_part * (int64_t)sizeof(double), false));
  N->cap_b = B;
  return KPM_OK;
}

static bool aligned16(const void* p, int ld) { return reinterpret_cast<uintptr_t>(p) % 16 == 0 && ld % 4 == 0; }
// A launch of n workgroups, rounded up to whole rounds over the eight XCDs.
static dim3 xcd_grid(int64_t n) { return dim3((unsigned)(ceil_div(n, 8) * 8)); }
// Output tiles of 32 nw x 32 nw.
static void set_tiles(Gemm& g, int nw) {
  g.tm = (int)ceil_div(g.M, 32 * nw);
  g.tn = (int)ceil_div(g.N, 32 * nw);
}
static bool vector_loads(const Gemm& g) { return aligned16(g.A, g.lda) && aligned16(g.B, g.ldb); }

// C = epilogue(A B), A [M][K], B [K][N].
template <int EPI, int NW, int CH>
static void gemm_forward_tiles(Gemm& g, hipStream_t s) {
  set_tiles(g, NW);
  auto fn = vector_loads(g) ? mlp_gemm<false, false, NW, EPI, true, false, CH> : mlp_gemm<false, false, NW, EPI, false, false, CH>;
  if constexpr (EPI == EPI_GELU) {
    if (g.x_shift)
      fn = vector_loads(g) ? mlp_gemm<false, false, NW, EPI, true, true, CH> : mlp_gemm<false, false, NW, EPI, false, true, CH>;
  }
  hipLaunchKernelGGL(fn, xcd_grid((int64_t)g.tm * g.tn), dim3(kGemmThreads), 0, s, g);
}
// Large batches: from 384 tiles of 64 x 64 on (one and a half per CU) the product is no
// longer bound by its chain but by how often the panels are read, and by the loads in
// flight where they are scalar: 64 x 64 tiles with stages of 32 indices (41 KB, three
// workgroups per CU).  FP32 inference, 32 x 32 tiles -> these: 256-1024-1792, batch 1024
// 111 -> 99 us, 65536 6084 -> 3778; 255-1023-1791 (scalar loads), 65536 10655 -> 5442;
// at 128 and 224 tiles a layer 67 -> 78, at 256 and 192 39 -> 43.  The sums run in the
// same order: same bits.
template <int EPI>
static void gemm_forward(Gemm& g, hipStream_t s) {
  if (ceil_div(g.M, 64) * ceil_div(g.N, 64) >= 384) gemm_forward_tiles<EPI, 2, 32>(g, s);
  else gemm_forward_tiles<EPI, 1, kChunk>(g, s);
}

static Gemm layer_gemm(kpm_mlp* N, const float* A, int ni, int layer, int no, int B) {
  Gemm g;
  g.A = A;
  g.lda = g.K = ni;
  g.B = N->par + N->off[2 * layer];
  g.ldb = g.ldc = g.N = no;
  g.bias = N->par + N->off[2 * layer + 1];
  g.M = B;
  return g;
}

// The hidden layers in FP32: pre-activations Z1, Z2, activations A1, A2.
static void forward_hidden(kpm_mlp* N, const float* X, int B, hipStream_t s) {
  Gemm g = layer_gemm(N, X, N->n_in, 0, N->n_hid, B);
  if (N->scaled) {
    g.x_shift = N->x_shift;
    g.x_scale = N->x_scale;
  }
  g.C = N->A1;
  g.Z = N->Z1;
  gemm_forward<EPI_GELU>(g, s);
  g = layer_gemm(N, N->A1, N->n_hid, 1, N->n_hid, B);
  g.C = N->A2;
  g.Z = N->Z2;
  gemm_forward<EPI_GELU>(g, s);
}

// The first n_cols columns of the network's output, in original units, into Y [B][n_out].
static void forward(kpm_mlp* N, const float* X, int B, bool bf16, float* Y, int n_cols, hipStream_t s) {
  const int ni = N->n_in, nh = N->n_hid, no = N->n_out;
  const float* xs = N->scaled ? N->x_shift : nullptr;
  const float* ys = N->scaled ? N->y_shift : nullptr;
  if (!bf16) {
    forward_hidden(N, X, B, s);
    Gemm g = layer_gemm(N, N->A2, nh, 2, no, B);
    g.N = n_cols;
    g.C = Y;
    g.y_shift = ys;
    g.y_scale = N->y_scale;
    gemm_forward<EPI_BIAS>(g, s);
    return;
  }
  const float* P = N->par;
  const int ldh = (int)ceil_div(nh, 32) * 32;
  const unsigned gm = (unsigned)ceil_div(B, 256);
  auto first = aligned16(X, ni) ? mlp_infer_kernel<1, true> : mlp_infer_kernel<0, true>;
  hipLaunchKernelGGL(first, dim3(ldh / 32, gm), dim3(kInferThreads), 0, s, X, ni, P + N->off[0], nh, P + N->off[1], B,
                     nh, ni, xs, N->x_scale, nullptr, nullptr, N->A1, ldh);
  hipLaunchKernelGGL((mlp_infer_kernel<2, true>), dim3(ldh / 32, gm), dim3(kInferThreads), 0, s, N->A1, ldh,
                     P + N->off[2], nh, P + N->off[3], B, nh, nh, nullptr, nullptr, nullptr, nullptr, N->A2, ldh);
  hipLaunchKernelGGL((mlp_infer_kernel<2, false>), dim3((unsigned)ceil_div(n_cols, 32), gm), dim3(kInferThreads), 0, s,
                     N->A2, ldh, P + N->off[4], no, P + N->off[5], B, n_cols, nh, nullptr, nullptr, ys, N->y_scale, Y,
                     no);
}

// Forward, loss (FP64, into *loss) and backward: the gradients into N->grad, or
// with ad one Adam step.  A layer's weights are updated once the gradient of
// the layer below no longer needs them.
template <int EPIW>
static void forward_backward_t(kpm_mlp* N, const float* X, const float* T, const float* w, int B, const AdamArgs* ad,
                               double* loss, hipStream_t s) {
  const int ni = N->n_in, nh = N->n_hid, no = N->n_out;
  forward_hidden(N, X, B, s);
  Gemm out = layer_gemm(N, N->A2, nh, 2, no, B);
  out.C = N->dY;
  out.T = T;
  out.w = w;
  out.partial = N->partial;
  if (N->scaled) {
    out.y_shift = N->y_shift;
    out.y_scale = N->y_scale;
  }
  gemm_forward<EPI_LOSS>(out, s);
  // dZ = (dOut W^T) gelu'(Z).
  auto act = [&](const float* dO, int n, int layer, const float* Z, float* dZ) {
    Gemm g;
    g.A = dO;
    g.B = N->par + N->off[2 * layer];
    g.lda = g.ldb = g.K = n;
    g.M = B;
    g.N = g.ldc = nh;
    g.Z = const_cast<float*>(Z);
    g.C = dZ;
    return g;
  };
  // dW = A^T dOut and the bias gradient of one layer.
  auto wgt = [&](const float* A, int rows, const float* dO, int cols, int layer) {
    Gemm g;
    g.A = A;
    g.lda = g.M = rows;
    g.B = dO;
    g.ldb = g.ldc = g.N = cols;
    g.K = B;
    const int64_t wo = N->off[2 * layer], bo = N->off[2 * layer + 1];
    g.C = N->grad + wo;
    g.bias_grad = N->grad + bo;
    g.par = N->par + wo;
    g.m = N->m + wo;
    g.v = N->v + wo;
    g.bpar = N->par + bo;
    g.bm = N->m + bo;
    g.bv = N->v + bo;
    if (ad) g.ad = *ad;
    set_tiles(g, 2);
    return g;
  };
  // The activation gradients' chains are as long as the widths: 32 x 32 tiles.  The
  // weight gradients' are as long as the batch, over many more outputs: 64 x 64.
  Gemm a2 = act(N->dY, no, 2, N->Z2, N->dZ2), a1 = act(N->dZ2, nh, 1, N->Z1, N->dZ1);
  Gemm w3 = wgt(N->A2, nh, N->dY, no, 2), w2 = wgt(N->A1, nh, N->dZ2, nh, 1), w1 = wgt(X, ni, N->dZ1, nh, 0);
  if (N->scaled) {
    w1.x_shift = N->x_shift;
    w1.x_scale = N->x_scale;
  }
  set_tiles(a2, 1);
  set_tiles(a1, 1);
  hipLaunchKernelGGL((vector_loads(a2) ? mlp_gemm<false, true, 1, EPI_GELU_BACK, true, false>
                                       : mlp_gemm<false, true, 1, EPI_GELU_BACK, false, false>),
                     xcd_grid((int64_t)a2.tm * a2.tn), dim3(kGemmThreads), 0, s, a2);
  hipLaunchKernelGGL((vector_loads(a1) && vector_loads(w3) ? mlp_back_pair<EPIW, true> : mlp_back_pair<EPIW, false>),
                     xcd_grid((int64_t)a1.tm * a1.tn + (int64_t)w3.tm * w3.tn), dim3(kGemmThreads), 0, s, a1, w3);
  const bool vec = vector_loads(w2) && vector_loads(w1);
  auto last = w1.x_shift ? (vec ? mlp_weight_pair<EPIW, true, true> : mlp_weight_pair<EPIW, false, true>)
                         : (vec ? mlp_weight_pair<EPIW, true, false> : mlp_weight_pair<EPIW, false, false>);
  hipLaunchKernelGGL(last,
                     xcd_grid((int64_t)w2.tm * w2.tn + (int64_t)w1.tm * w1.tn + 1), dim3(kGemmThreads), 0, s, w2, w1,
                     N->partial, out.tm * out.tn, loss);
}

static void forward_backward(kpm_mlp* N, const float* X, const float* T, const float* w, int B, const AdamArgs* ad,
                             double* loss, hipStream_t s) {
  if (ad) forward_backward_t<EPI_ADAM>(N, X, T, w, B, ad, loss, s);
  else forward_backward_t<EPI_GRAD>(N, X, T, w, B, nullptr, loss, s);
}

}  // namespace kpm

extern "C" {

int kpm_mlp_create(int32_t n_in, int32_t n_hidden, int32_t n_out, uint64_t seed, kpm_mlp_t** out) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(out != nullptr, "NULL output");
  *out = nullptr;
  KPM_CHECK_ARG(n_in >= 1 && n_hidden >= 1 && n_out >= 1 && n_in <= 65536 && n_hidden <= 65536 && n_out <= 65536,
                "layer sizes must be in [1, 65536]");
  kpm_mlp* N = new (std::nothrow) kpm_mlp();
  if (!N) {
    set_error("kpm_mlp_create: out of host memory");
    return KPM_E_NOMEM;
  }
  N->n_in = n_in;
  N->n_hid = n_hidden;
  N->n_out = n_out;
  const int64_t sz[6] = {(int64_t)n_in * n_hidden, n_hidden, (int64_t)n_hidden * n_hidden, n_hidden,
                         (int64_t)n_hidden * n_out, n_out};
  int64_t o = 0;
  for (int i = 0; i < 6; ++i) {
    N->off[i] = o;
    o += (sz[i] + 63) / 64 * 64;
  }
  N->n_par = o;
  hipError_t e = ::kpm::dev_malloc(&N->par, o * 4, false);
  if (e == hipSuccess) e = ::kpm::dev_malloc(&N->grad, o * 4, false);
  if (e == hipSuccess) e = ::kpm::dev_malloc(&N->m, o * 4, false);
  if (e == hipSuccess) e = ::kpm::dev_malloc(&N->v, o * 4, false);
  if (e == hipSuccess) e = ::kpm::dev_malloc(&N->loss_dev, sizeof(double), false);
  if (e == hipSuccess) {
    const unsigned gb = (unsigned)ceil_div(o, 256);
    hipLaunchKernelGGL(fill_f32, dim3(gb), dim3(256), 0, 0, N->par, o, 0.f);
    hipLaunchKernelGGL(fill_f32, dim3(gb), dim3(256), 0, 0, N->grad, o, 0.f);
    hipLaunchKernelGGL(fill_f32, dim3(gb), dim3(256), 0, 0, N->m, o, 0.f);
    hipLaunchKernelGGL(fill_f32, dim3(gb), dim3(256), 0, 0, N->v, o, 0.f);
    const int fan[3] = {n_in, n_hidden, n_hidden};
    for (int l = 0; l < 3; ++l) {
      const int64_t n = sz[2 * l];
      hipLaunchKernelGGL(init_uniform_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, 0, N->par + N->off[2 * l],
                         n, sm_key(5, seed, (uint64_t)l, 0), (float)std::sqrt(3.0 / fan[l]));
    }
    e = ::kpm::launch_status();
    if (e == hipSuccess) e = hipDeviceSynchronize();
  }
  if (e != hipSuccess) {
    set_error("kpm_mlp_create: %s", hipGetErrorString(e));
    kpm_mlp_destroy(N);
    return e == hipErrorOutOfMemory ? KPM_E_NOMEM : KPM_E_DEVICE;
  }
  *out = N;
  return KPM_OK;
}

int kpm_mlp_destroy(kpm_mlp_t* N) {
  if (!N) return KPM_OK;
  void* bufs[] = {N->par, N->grad, N->m, N->v, N->Z1, N->A1, N->Z2, N->A2, N->Y, N->dY, N->dZ1, N->dZ2, N->partial,
                  N->loss_dev, N->x_shift, N->x_scale, N->y_shift, N->y_scale};
  for (void* b : bufs)
    if (b) (void)::kpm::dev_free(b);
  delete N;
  return KPM_OK;
}

int kpm_mlp_num_params(const kpm_mlp_t* N, int64_t* n) {
  using namespace kpm;
  KPM_CHECK_ARG(N && n, "NULL argument");
  *n = (int64_t)N->n_in * N->n_hid + N->n_hid + (int64_t)N->n_hid * N->n_hid + N->n_hid +
       (int64_t)N->n_hid * N->n_out + N->n_out;
  return KPM_OK;
}

// Parameters / gradients exchanged in packed order W1 [n_in][n_hid], b1, W2 [n_hid][n_hid], b2, W3 [n_hid][n_out], b3.
static int mlp_copy(kpm_mlp_t* N, float* dev_base, float* host, bool to_host) {
  using namespace kpm;
  const int64_t sz[6] = {(int64_t)N->n_in * N->n_hid, N->n_hid, (int64_t)N->n_hid * N->n_hid, N->n_hid,
                         (int64_t)N->n_hid * N->n_out, N->n_out};
  int64_t h = 0;
  for (int i = 0; i < 6; ++i) {
    if (to_host) KPM_TRY_HIP(hipMemcpy(host + h, dev_base + N->off[i], sz[i] * 4, hipMemcpyDeviceToHost));
    else KPM_TRY_HIP(hipMemcpy(dev_base + N->off[i], host + h, sz[i] * 4, hipMemcpyHostToDevice));
    h += sz[i];
  }
  return KPM_OK;
}

int kpm_mlp_get_params(kpm_mlp_t* N, float* params) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && params, "NULL argument");
  KPM_TRY_SYNC(hipDeviceSynchronize());
  return mlp_copy(N, N->par, params, true);
}

int kpm_mlp_set_params(kpm_mlp_t* N, const float* params) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && params, "NULL argument");
  KPM_TRY_SYNC(hipDeviceSynchronize());
  N->t = 0;
  const unsigned gb = (unsigned)ceil_div(N->n_par, 256);
  hipLaunchKernelGGL(fill_f32, dim3(gb), dim3(256), 0, 0, N->m, N->n_par, 0.f);
  hipLaunchKernelGGL(fill_f32, dim3(gb), dim3(256), 0, 0, N->v, N->n_par, 0.f);
  KPM_TRY_SYNC(hipDeviceSynchronize());
  return mlp_copy(N, N->par, const_cast<float*>(params), false);
}

int kpm_mlp_forward(kpm_mlp_t* N, const float* x, int32_t batch, float* y, int32_t use_bf16, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && x && y && batch >= 1, "bad arguments");
  KPM_TRY(mlp_reserve(N, batch));
  forward(N, x, batch, use_bf16 != 0, y, N->n_out, (hipStream_t)hip_stream);
  KPM_TRY_HIP(hipGetLastError());
  return KPM_OK;
}

int kpm_mlp_rel_error(kpm_mlp_t* N, const float* x, const double* ref, const float* weights, int32_t batch,
                      int32_t n_cmp, int32_t use_bf16, double* err, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && x && ref && weights && err && batch >= 1, "bad arguments");
  KPM_CHECK_ARG(n_cmp >= 1 && n_cmp <= N->n_out, "n_cmp must be in [1, n_out]");
  KPM_TRY(mlp_reserve(N, batch));
  hipStream_t s = (hipStream_t)hip_stream;
  forward(N, x, batch, use_bf16 != 0, N->Y, n_cmp, s);   // the compared columns only
  hipLaunchKernelGGL(rel_error_kernel, dim3(batch), dim3(256), 0, s, N->Y, N->n_out, ref, n_cmp, weights,
                     (const double*)nullptr, err);
  KPM_TRY_HIP(hipGetLastError());
  return KPM_OK;
}

int kpm_mlp_noise_z(kpm_mlp_t* N, const float* x, const double* ref, const double* noise, const float* weights,
                    int32_t batch, int32_t n_cmp, int32_t use_bf16, double* z, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && x && ref && noise && weights && z && batch >= 1, "bad arguments");
  KPM_CHECK_ARG(n_cmp >= 1 && n_cmp <= N->n_out, "n_cmp must be in [1, n_out]");
  KPM_TRY(mlp_reserve(N, batch));
  hipStream_t s = (hipStream_t)hip_stream;
  forward(N, x, batch, use_bf16 != 0, N->Y, n_cmp, s);   // the compared columns only
  hipLaunchKernelGGL(rel_error_kernel, dim3(batch), dim3(256), 0, s, N->Y, N->n_out, ref, n_cmp, weights, noise, z);
  KPM_TRY_HIP(hipGetLastError());
  return KPM_OK;
}

int kpm_mlp_eval_loss(kpm_mlp_t* N, const float* x, const float* target, const float* weights, int32_t batch,
                      int32_t use_bf16, double* loss_dev_out, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && x && target && weights && loss_dev_out && batch >= 1, "bad arguments");
  KPM_TRY(mlp_reserve(N, batch));
  hipStream_t s = (hipStream_t)hip_stream;
  forward(N, x, batch, use_bf16 != 0, N->Y, N->n_out, s);
  hipLaunchKernelGGL(mlp_loss_kernel, dim3(kLossBlocks), dim3(256), 0, s, N->Y, target, weights, batch, N->n_out,
                     N->partial);
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, s, N->partial, kLossBlocks, loss_dev_out);
  KPM_TRY_HIP(hipGetLastError());
  return KPM_OK;
}

int kpm_mlp_fit_scaling(kpm_mlp_t* N, const float* x, const float* target, int64_t n_rows, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && x && target && n_rows >= 1, "bad arguments");
  hipStream_t s = (hipStream_t)hip_stream;
  // Each buffer on its own, so that a call after a failed allocation completes the set.
  if (!N->x_shift) KPM_TRY_HIP(::kpm::dev_malloc(&N->x_shift, N->n_in * 4, false));
  if (!N->x_scale) KPM_TRY_HIP(::kpm::dev_malloc(&N->x_scale, N->n_in * 4, false));
  if (!N->y_shift) KPM_TRY_HIP(::kpm::dev_malloc(&N->y_shift, N->n_out * 4, false));
  if (!N->y_scale) KPM_TRY_HIP(::kpm::dev_malloc(&N->y_scale, N->n_out * 4, false));
  hipLaunchKernelGGL(column_stats_kernel, dim3((unsigned)ceil_div(N->n_in, kStatCols)), dim3(1024), 0, s, x, n_rows,
                     N->n_in, N->x_shift, N->x_scale);
  hipLaunchKernelGGL(column_stats_kernel, dim3((unsigned)ceil_div(N->n_out, kStatCols)), dim3(1024), 0, s, target,
                     n_rows, N->n_out, N->y_shift, N->y_scale);
  KPM_TRY_HIP(hipGetLastError());
  KPM_TRY_SYNC(hipStreamSynchronize(s));
  N->scaled = true;
  return KPM_OK;
}

int kpm_mlp_gradients(kpm_mlp_t* N, const float* x, const float* target, const float* weights, int32_t batch,
                      float* grads_host, double* loss, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && x && target && weights && batch >= 1, "bad arguments");
  KPM_TRY(mlp_reserve(N, batch));
  hipStream_t s = (hipStream_t)hip_stream;
  forward_backward(N, x, target, weights, batch, nullptr, N->loss_dev, s);
  KPM_TRY_HIP(hipGetLastError());
  KPM_TRY_SYNC(hipStreamSynchronize(s));
  if (loss) KPM_TRY_HIP(hipMemcpy(loss, N->loss_dev, sizeof(double), hipMemcpyDeviceToHost));
  if (grads_host) KPM_TRY(mlp_copy(N, N->grad, grads_host, true));
  return KPM_OK;
}

int kpm_mlp_train_step(kpm_mlp_t* N, const float* x, const float* target, const float* weights, int32_t batch,
                       float lr, double* loss_dev_out, void* hip_stream) {
  using namespace kpm;
  clear_error();
  KPM_CHECK_ARG(N && x && target && weights && batch >= 1, "bad arguments");
  KPM_CHECK_ARG(lr > 0.f && std::isfinite(lr), "lr must be > 0");
  KPM_TRY(mlp_reserve(N, batch));
  hipStream_t s = (hipStream_t)hip_stream;
  N->t += 1;
  AdamArgs ad;
  ad.lr = lr;
  ad.c1 = (float)(1.0 / (1.0 - std::pow(kBeta1, (double)N->t)));
  ad.c2 = (float)(1.0 / (1.0 - std::pow(kBeta2, (double)N->t)));
  forward_backward(N, x, target, weights, batch, &ad, loss_dev_out ? loss_dev_out : N->loss_dev, s);
  KPM_TRY_HIP(hipGetLastError());
  return KPM_OK;
}

}  // extern "C"
