// Learned surrogate of the moment -> transmittance reconstruction: a
// 7 -> 64 -> 64 -> 1 MLP (tanh-GELU hidden layers, sigmoid output F, optical
// depth m_0 F) with bf16 weights and activations and fp32 accumulation.
//
// Every layer is a dense contraction and runs on the matrix cores
// (v_mfma_f32_32x32x16_bf16), a tile of 32 queries per wave, as the transposed
// products (weights times activations):
//   layer 1  Z1^T[64x32] = W1p X^T,   X = (x_hi, x_lo) split of the 7 fp32
//            inputs into bf16 pairs (W1p repeats W1 for both halves), so the
//            inputs keep ~16 mantissa bits;
//   layer 2  Z2^T[64x32] = W2 H1^T,   H1 = bf16(GELU(Z1 + b1));
//   layer 3  out = GELU(Z2 + b2) . w3 + b3, summed in neuron order;
// and the training step adds dH1^T = W2^T dZ2^T, dW2 = dZ2^T H1 and dW1 = dZ1^T X.
// MFMA operand layout (wave64, 32x32x16): lane l holds A[l % 32][8 (l / 32) + e]
// and B[8 (l / 32) + e][l % 32], e = 0..7, and accumulator element r of lane l is
// C[8 (r / 4) + 4 (l / 32) + r % 4][l % 32].
#include "kernels.h"

namespace mb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kH = 64;       // hidden width
constexpr int kIn = 7;       // inputs: 6 moment features + query
constexpr int kXStride = 16; // bf16 per input row (hi 0..6, lo 7..13, 0 pad)
// flat fp32 parameter vector theta
constexpr int O_W1 = 0;              // [64][7]
constexpr int O_B1 = O_W1 + kH * kIn; // [64]
constexpr int O_W2 = O_B1 + kH;       // [64][64] (out, in)
constexpr int O_B2 = O_W2 + kH * kH;  // [64]
constexpr int O_W3 = O_B2 + kH;       // [64]
constexpr int O_B3 = O_W3 + kH;       // [1]
constexpr int kParams = O_B3 + 1;     // 4737
// layout of a row of partial gradients (dW1 kept unfolded over the hi/lo halves)
constexpr int Q_W1 = 0;               // [64][16]
constexpr int Q_B1 = Q_W1 + kH * 16;
constexpr int Q_W2 = Q_B1 + kH;
constexpr int Q_B2 = Q_W2 + kH * kH;
constexpr int Q_W3 = Q_B2 + kH;
constexpr int Q_B3 = Q_W3 + kH;
constexpr int Q_LOSS = Q_B3 + 1;
constexpr int kPartial = Q_LOSS + 3;  // padded to a multiple of 4

struct MlpPacked {
  uint16_t w1[kH][kXStride];  // bf16 [n][k]: cols 0..6 = W1, 7..13 = W1, 14..15 = 0
  uint16_t w2[kH][kH];        // bf16 [n][k]
  uint16_t w2t[kH][kH];       // bf16 [k][n]
  float w3[kH];               // bf16-rounded
  float b1[kH], b2[kH];
  float b3;
  float pad[63];
  float w1f[kIn][kH];         // bf16-rounded W1 as fp32, [k][n] (input gradient)
};
static_assert(sizeof(MlpPacked) % 16 == 0, "packed weights must be 16-byte sized");

__host__ __device__ inline uint16_t bf16_bits(float x) {
  uint32_t u;
  memcpy(&u, &x, 4);
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even
  return (uint16_t)(u >> 16);
}
__host__ __device__ inline float bf16_float(uint16_t b) {
  uint32_t u = ((uint32_t)b) << 16;
  float f;
  memcpy(&f, &u, 4);
  return f;
}

__device__ __forceinline__ float gelu_d(float x, float& d) {
  // tanh form 0.5 x (1 + tanh(u)), u = c (x + a x^3), evaluated as x s with
  // s = 1 / (1 + exp(-2u)) (the same function: 0.5 (1 + tanh u) = s):
  // one exp2 and one reciprocal, no tanh
  const float c = 0.7978845608028654f, a = 0.044715f;
  const float k = -2.f * c * 1.4426950408889634f;  // -2 c log2(e)
  const float x2 = x * x;
  const float e = __builtin_amdgcn_exp2f(k * x * (1.f + a * x2));
  const float sg = fast_rcp(1.f + e);
  d = sg + 2.f * c * x * sg * (1.f - sg) * (1.f + 3.f * a * x2);
  return x * sg;
}
__device__ __forceinline__ bf16x8 lds_bf16x8(const uint16_t* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int c_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// ---------------------------------------------------------------------------
// Bound by its launch: 16 blocks, one element a thread and array.
__global__ __launch_bounds__(256) void k_mlp_pack(const float* th, MlpPacked* p) {
  const int t0 = blockIdx.x * blockDim.x + threadIdx.x, dt = gridDim.x * blockDim.x;
  for (int i = t0; i < kH * kXStride; i += dt) {
    int n = i / kXStride, k = i % kXStride;
    float v = k < kIn ? th[O_W1 + n * kIn + k] : (k < 2 * kIn ? th[O_W1 + n * kIn + k - kIn] : 0.f);
    p->w1[n][k] = bf16_bits(v);
  }
  for (int i = t0; i < kH * kH; i += dt) {
    int n = i / kH, k = i % kH;
    uint16_t b = bf16_bits(th[O_W2 + i]);
    p->w2[n][k] = b;
    p->w2t[k][n] = b;
  }
  for (int i = t0; i < kH; i += dt) {
    p->w3[i] = bf16_float(bf16_bits(th[O_W3 + i]));
    p->b1[i] = th[O_B1 + i];
    p->b2[i] = th[O_B2 + i];
  }
  if (t0 == 0) p->b3 = th[O_B3];
  for (int i = t0; i < 63; i += dt) p->pad[i] = 0.f;
  for (int i = t0; i < kH * kIn; i += dt) {
    int n = i / kIn, k = i % kIn;
    p->w1f[k][n] = bf16_float(bf16_bits(th[O_W1 + i]));
  }
}

__device__ __forceinline__ float sigmoid(float x) { return fast_rcp(1.f + __expf(-x)); }

// ---------------------------------------------------------------------------
// The activations stay in registers from layer to layer (inference takes two tiles
// of 32 queries a wave and step): lane l holds the column of query l % 32, accumulator element r its neuron 8 (r / 4) +
// 4 (l / 32) + r % 4. Rounded to bf16 pairs, eight consecutive elements of a
// lane are half a k-block of the next layer's B operand; exchanging the middle
// quarters between the wave's halves (permlane32_swap) puts them in the operand's
// order, so H1 never visits LDS. The weights stay in registers for all of a
// wave's queries. Each product and sum keeps the order of the row-wise form, so
// the outputs do not depend on the form.
//
// Bound by the GELUs on the vector unit: 64 evaluations of about 34 issue cycles
// per lane and tile (16 of them the two transcendentals), of 2700 a tile in all,
// beside 10 matrix instructions of 32 cycles on the matrix pipe. Measured, with
// H1 and the weights passed through LDS before: 68.4 M nodes of tables
// 3.95 -> 3.05 ms, the query list of a surrogate step (960 x 540) 581 -> 462 us.
// Two to four waves a SIMD and one or two tiles a step time alike within 5%.
// ---------------------------------------------------------------------------
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));  // nearest even
}
// a's upper half-wave changes places with b's lower one
__device__ __forceinline__ void swap_halves(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  uint32_t u = __float_as_uint(a), v = __float_as_uint(b);
  swap_halves(u, v);
  a = __uint_as_float(u);
  b = __uint_as_float(v);
}

struct RegWeights {
  bf16x8 w1[2], w2[2][4];  // A operands: neurons 32 t + l % 32, k-block
};

__device__ __forceinline__ bf16x8 global_bf16x8(const uint16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

__device__ __forceinline__ RegWeights load_weights(const MlpPacked* P, int lane) {
  RegWeights w;
  const int lr = lane & 31, hk = 8 * (lane >> 5);
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    w.w1[t] = global_bf16x8(&P->w1[32 * t + lr][hk]);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) w.w2[t][kt] = global_bf16x8(&P->w2[32 * t + lr][16 * kt + hk]);
  }
  return w;
}

// B operand of layer 1 for this lane's query (its kIn inputs v): k = 0..6 the
// bf16 values, 7..13 what they leave of the inputs, 14, 15 zero
__device__ __forceinline__ bf16x8 input_operand(const float* v, int lane) {
  float lo[kIn];
  uint32_t hi[4];
#pragma unroll
  for (int k = 0; k < kIn; k += 2) {
    const float v1 = k + 1 < kIn ? v[k + 1] : 0.f;
    hi[k / 2] = pack_bf16(v[k], v1);
    lo[k] = v[k] - __uint_as_float(hi[k / 2] << 16);
    if (k + 1 < kIn) lo[k + 1] = v1 - __uint_as_float(hi[k / 2] & 0xffff0000u);
  }
  const uint32_t l0 = pack_bf16(lo[0], 0.f);
  const bool up = lane >= 32;
  uint4 o;
  o.x = up ? pack_bf16(lo[1], lo[2]) : hi[0];
  o.y = up ? pack_bf16(lo[3], lo[4]) : hi[1];
  o.z = up ? pack_bf16(lo[5], lo[6]) : hi[2];
  o.w = up ? 0u : (hi[3] | (l0 << 16));
  return __builtin_bit_cast(bf16x8, o);
}

// the bf16 B operands of the next product from this lane's 64-neuron column
// z[2] (elements as above)
__device__ __forceinline__ void column_operand(const f32x16* z, bf16x8* op) {
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      uint4 o;
      o.x = pack_bf16(z[t][8 * s + 0], z[t][8 * s + 1]);
      o.y = pack_bf16(z[t][8 * s + 2], z[t][8 * s + 3]);
      o.z = pack_bf16(z[t][8 * s + 4], z[t][8 * s + 5]);
      o.w = pack_bf16(z[t][8 * s + 6], z[t][8 * s + 7]);
      swap_halves(o.x, o.z);
      swap_halves(o.y, o.w);
      op[2 * t + s] = __builtin_bit_cast(bf16x8, o);
    }
}

// Layers 1 and 2 of a tile's 32 queries and the terms of layer 3: s[r] = the
// output terms of neurons n and n + 32 for n = 8 (r / 4) + 4 (l / 32) + r % 4.
// KEEP 1: d1, d2 receive GELU' at the two layers; 2: also h1 the bf16 operand of
// layer 2 and h2 the activations of layer 2.
struct RowConsts {
  float b1[kH], b2[kH], w3[kH];
};
template <int KEEP>
__device__ __forceinline__ void mlp_tile(const RegWeights& w, const RowConsts& c, bf16x8 x, int lane, float* s,
                                         f32x16* d1 = nullptr, f32x16* d2 = nullptr, bf16x8* h1 = nullptr,
                                         f32x16* h2 = nullptr) {
  const int h4 = 4 * (lane >> 5);
  f32x16 z[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    z[t] = mfma(w.w1[t], x, f32x16{});
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 b = *reinterpret_cast<const float4*>(&c.b1[32 * t + 8 * g + h4]);
      const float bb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float d;
        z[t][4 * g + j] = gelu_d(z[t][4 * g + j] + bb[j], d);
        if constexpr (KEEP > 0) d1[t][4 * g + j] = d;
      }
    }
  }
  bf16x8 op[4];
  column_operand(z, op);
  if constexpr (KEEP > 1)
#pragma unroll
    for (int k = 0; k < 4; ++k) h1[k] = op[k];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    z[t] = f32x16{};
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) z[t] = mfma(w.w2[t][kt], op[kt], z[t]);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 b = *reinterpret_cast<const float4*>(&c.b2[32 * t + 8 * g + h4]);
      const float4 q = *reinterpret_cast<const float4*>(&c.w3[32 * t + 8 * g + h4]);
      const float bb[4] = {b.x, b.y, b.z, b.w}, qq[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float d;
        const float a = gelu_d(z[t][4 * g + j] + bb[j], d);
        if constexpr (KEEP > 0) d2[t][4 * g + j] = d;
        if constexpr (KEEP > 1) h2[t][4 * g + j] = a;
        s[4 * g + j] = t == 0 ? a * qq[j] : fmaf(a, qq[j], s[4 * g + j]);
      }
    }
}

// the output pre-activation from a query's 32 terms in neuron order: lo[r] of the
// neurons with an even quarter, hi[r] of the others
__device__ __forceinline__ float sum_terms(float b3, const float* lo, const float* hi) {
  float out = b3;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int j = 0; j < 4; ++j) out += lo[4 * g + j];
#pragma unroll
    for (int j = 0; j < 4; ++j) out += hi[4 * g + j];
  }
  return out;
}

__device__ __forceinline__ void stage_consts(RowConsts& c, const MlpPacked* P) {
  for (int i = threadIdx.x; i < kH; i += blockDim.x) {
    c.b1[i] = P->b1[i];
    c.b2[i] = P->b2[i];
    c.w3[i] = P->w3[i];
  }
  __syncthreads();
}

// F of the n queries, 64 a wave and step. A source (q, step) stands at query q,
// loads its inputs (zeros beyond the list) and moves on by step; load returns
// whether the query's output is wanted. A step none of whose outputs is writes none.
template <class Source, class Output>
__device__ __forceinline__ void mlp_queries(const MlpPacked* P, int64_t n, const Source& src, Output&& output) {
  __shared__ __align__(16) RowConsts c;
  stage_consts(c, P);
  const int lane = threadIdx.x & 63, lr = lane & 31;
  const RegWeights w = load_weights(P, lane);
  const float b3 = P->b3;
  const int64_t step = (int64_t)gridDim.x * (blockDim.x >> 6) * 64;
  int64_t q0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64;
  if (q0 >= n) return;
  Source in[2] = {src, src};
  float v[2][kIn];
  in[0].start(q0 + lr, step);
  in[1].start(q0 + 32 + lr, step);
  auto load = [&]() __attribute__((always_inline)) {
    const bool w0 = in[0].load(v[0]), w1 = in[1].load(v[1]);
    return __ballot(w0 || w1) != 0;
  };
  bool wanted = load();
  for (; q0 < n; q0 += step) {
    const bool now = wanted;
    const bf16x8 x[2] = {input_operand(v[0], lane), input_operand(v[1], lane)};
    if (q0 + step < n) {  // the next step's inputs load behind this one's arithmetic
      in[0].advance();
      in[1].advance();
      wanted = load();
    }
    if (!now) continue;
    float s[2][16];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      asm volatile("" ::: "memory");  // the constants are read anew, not kept in 96 registers
      mlp_tile<0>(w, c, x[t], lane, s[t]);
    }
    // tile 0's queries to the lower half-wave, tile 1's to the upper
#pragma unroll
    for (int r = 0; r < 16; ++r) swap_halves(s[0][r], s[1][r]);
    const int64_t q = q0 + lane;
    const float f = sigmoid(sum_terms(b3, s[0], s[1]));
    if (q < n) output(q, f);
  }
}

struct RowSource {  // x [n][8]: a fit's rows
  const float* x;
  int64_t n, q = 0, by = 0;
  __device__ RowSource(const float* x_, int64_t n_) : x(x_), n(n_) {}
  __device__ __forceinline__ void start(int64_t q_, int64_t step) {
    q = q_;
    by = step;
  }
  __device__ __forceinline__ void advance() { q += by; }
  __device__ __forceinline__ bool load(float* v) const {
    const bool valid = q < n;
    const float* r = x + (valid ? q : 0) * 8;
#pragma unroll
    for (int k = 0; k < kIn; ++k) v[k] = valid ? r[k] : 0.f;
    return true;
  }
};

// the render's query list: the six features of pixel pix[q] (slots of a list that
// overflowed may hold no query: their pixel index is kept inside the image, their
// outputs are never read) and the standardised query z[q]
struct GatherSource {
  const float* feat;
  const int* pix;
  const float* z;
  int64_t n_pix, n, q = 0, by = 0;
  __device__ GatherSource(const float* feat_, const int* pix_, const float* z_, int64_t n_pix_, int64_t n_)
      : feat(feat_), pix(pix_), z(z_), n_pix(n_pix_), n(n_) {}
  __device__ __forceinline__ void start(int64_t q_, int64_t step) {
    q = q_;
    by = step;
  }
  __device__ __forceinline__ void advance() { q += by; }
  __device__ __forceinline__ bool load(float* v) const {
    const bool valid = q < n;
    int64_t p = valid ? (int64_t)pix[q] : 0;
    p = (p >= 0 && p < n_pix) ? p : 0;
    const float* f = feat + p * kPixFeat;
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = valid ? f[k] : 0.f;
    v[6] = valid ? z[q] : 0.f;
    return true;
  }
};

// the nodes of every pixel's table: entry q = p n_nodes + g takes the features of
// pixel p and the standardised query -kTabZ + g 2 kTabZ / (n_nodes - 1)
struct TableSource {
  const float* feat;
  int64_t n_pix, p = 0, dp = 0;
  int n_nodes, g = 0, dg = 0;
  float dz;
  __device__ TableSource(const float* feat_, int64_t n_pix_, int n_nodes_)
      : feat(feat_), n_pix(n_pix_), n_nodes(n_nodes_), dz(2.f * kTabZ / (float)(n_nodes_ - 1)) {}
  __device__ __forceinline__ void start(int64_t q, int64_t step) {
    p = q / n_nodes;
    g = (int)(q - p * n_nodes);
    dp = step / n_nodes;
    dg = (int)(step - dp * n_nodes);
  }
  __device__ __forceinline__ void advance() {
    p += dp;
    g += dg;
    if (g >= n_nodes) {
      g -= n_nodes;
      ++p;
    }
  }
  __device__ __forceinline__ bool load(float* v) const {
    const bool valid = p < n_pix;
    const float* f = feat + (valid ? p : 0) * kPixFeat;
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = valid ? f[k] : 0.f;
    v[6] = -kTabZ + dz * (float)g;
    return valid && f[6] > 0.f;  // no optical depth: an empty pixel, whose table is never read
  }
};

__global__ __launch_bounds__(256, 3) void k_mlp_forward(const MlpPacked* P, const float* x, int64_t n, float* f_out) {
  mlp_queries(P, n, RowSource(x, n), [&](int64_t q, float f) __attribute__((always_inline)) { f_out[q] = f; });
}

// The number of queries is read on the device (the render pass appends them).
__global__ __launch_bounds__(256, 3) void k_mlp_forward_gather(const MlpPacked* P, const float* pixfeat,
                                                               const int* q_pix, const float* q_z,
                                                               const unsigned long long* q_count, int64_t q_cap,
                                                               int64_t n_pix, float* f_out) {
  const unsigned long long cnt = *q_count;
  const int64_t n = cnt < (unsigned long long)q_cap ? (int64_t)cnt : q_cap;
  mlp_queries(P, n, GatherSource(pixfeat, q_pix, q_z, n_pix, n),
              [&](int64_t q, float f) __attribute__((always_inline)) { f_out[q] = f; });
}

// tab [n_pix][n_nodes]: the tabulated schedule's F, for the pixels with an optical
// depth (54% in the case tabulated_network of perf/cases.py: 3.05 -> 1.84 ms)
__global__ __launch_bounds__(256, 3) void k_mlp_table(const MlpPacked* P, const float* pixfeat, int64_t n_pix,
                                                      int n_nodes, float* tab) {
  mlp_queries(P, n_pix * n_nodes, TableSource(pixfeat, n_pix, n_nodes),
              [&](int64_t q, float f) __attribute__((always_inline)) { tab[q] = f; });
}

// F and its gradient dF/dx with respect to the 7 inputs for every query of
// the render's list (for the backward pass through the surrogate): the forward
// tile with its GELU' kept, then dZ2 = F (1 - F) w3 GELU'(Z2) (bf16) against W2
// and dZ1 = dH1 GELU'(Z1) (bf16) against W1 as the forward's transposed products;
// W1's operand has an empty row first, so that the lower half-wave ends with
// (0, dx_0..2) and the upper with dx_3..6. out: [cap][8] = F, dF/dx_0..6.
// Bound by vector issue, 4360 cycles per 32 queries (GELU' adds 8 fused operations
// to each GELU): 2277 -> 848 us for the queries of a surrogate step (960 x 540),
// where the activations and both layers' products passed through LDS before and
// each GELU was evaluated twice; 1062 us with dx = dZ1 W1 on the vector unit, whose
// rounding error is 1.8 times the matrix instruction's (rms, 64 random terms).
__global__ __launch_bounds__(256, 2) void k_mlp_input_grad_gather(const MlpPacked* P, const float* pixfeat,
                                                               const int* q_pix, const float* q_z,
                                                               const unsigned long long* q_count, int64_t q_cap,
                                                               int64_t n_pix, float* out_g) {
  __shared__ __align__(16) RowConsts c;
  __shared__ __align__(16) uint16_t w2t[kH][kH + 8];  // W2^T, rows apart in the banks
  const unsigned long long cnt = *q_count;
  const int64_t n = cnt < (unsigned long long)q_cap ? (int64_t)cnt : q_cap;
  for (int i = threadIdx.x; i < kH * kH / 8; i += blockDim.x)
    *reinterpret_cast<bf16x8*>(&w2t[i / 8][8 * (i % 8)]) = global_bf16x8(&P->w2t[i / 8][8 * (i % 8)]);
  stage_consts(c, P);
  const int lane = threadIdx.x & 63, lr = lane & 31, half = lane >> 5;
  const RegWeights w = load_weights(P, lane);
  // W1^T as the A operand: row 0 empty, rows 1..7 the inputs
  bf16x8 w1t[4];
#pragma unroll
  for (int kt = 0; kt < 4; ++kt) {
    uint32_t u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float* f = &P->w1f[lr >= 1 && lr <= kIn ? lr - 1 : 0][16 * kt + 8 * half + 2 * j];
      u[j] = lr >= 1 && lr <= kIn ? pack_bf16(f[0], f[1]) : 0u;
    }
    w1t[kt] = __builtin_bit_cast(bf16x8, make_uint4(u[0], u[1], u[2], u[3]));
  }
  const float b3 = P->b3;
  const int64_t step = (int64_t)gridDim.x * (blockDim.x >> 6) * 32;
  int64_t q0 = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 32;
  if (q0 >= n) return;
  GatherSource in(pixfeat, q_pix, q_z, n_pix, n);
  float v[kIn];
  in.start(q0 + lr, step);
  in.load(v);
  for (; q0 < n; q0 += step) {
    const bf16x8 x = input_operand(v, lane);
    if (q0 + step < n) {
      in.advance();
      in.load(v);
    }
    float s[16], t[16];
    f32x16 d1[2], d2[2];
    asm volatile("" ::: "memory");  // the constants are read anew, not kept in registers
    mlp_tile<1>(w, c, x, lane, s, d1, d2);
#pragma unroll
    for (int r = 0; r < 16; ++r) {  // both halves end with all of the query's terms
      t[r] = s[r];
      swap_halves(s[r], t[r]);
    }
    const float f = sigmoid(sum_terms(b3, s, t));
    const float dout = f * (1.f - f);
    // dZ2, then dH1^T = W2^T dZ2^T
    f32x16 dz[2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 q = *reinterpret_cast<const float4*>(&c.w3[32 * m + 8 * g + 4 * half]);
        const float qq[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) dz[m][4 * g + j] = dout * qq[j] * d2[m][4 * g + j];
      }
    bf16x8 op[4];
    column_operand(dz, op);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      dz[m] = f32x16{};
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) dz[m] = mfma(lds_bf16x8(&w2t[32 * m + lr][16 * kt + 8 * half]), op[kt], dz[m]);
    }
    // dZ1 (bf16), dx^T = W1^T dZ1^T
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) dz[m][r] *= d1[m][r];
    column_operand(dz, op);
    f32x16 gx = {};
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) gx = mfma(w1t[kt], op[kt], gx);
    const int64_t q = q0 + lr;
    if (q < n) reinterpret_cast<float4*>(out_g + q * 8)[half] = make_float4(half ? gx[0] : f, gx[1], gx[2], gx[3]);
  }
}

// Forward + backward of the loss mean_q (exp(-m0 F) - t)^2 over the n queries of x
// [n][8] (7 inputs, m0): each block writes one row of partial gradients.
//
// The forward tile with GELU', H1 and GELU(Z2) kept, dZ2 = dout w3 GELU'(Z2) and
// dZ1 = dH1 GELU'(Z1) in the same layout (a lane per query), the bias and w3
// gradients summed per lane in fp32. The weight gradients contract over the
// queries: H1, dZ2, dZ1 and X pass through LDS once, transposed, and accumulate
// in registers (80 a lane) over all of a wave's tiles. One wave a SIMD, 512
// registers. Bound by latency at a batch of 65536 (two tiles of 5300 issue cycles a
// wave, its weights before and its sums after them): 94 -> 28 us, where each wave
// took 64 queries through LDS between all products, evaluated each GELU twice and
// spilled 182 registers.
constexpr int kTrainWaves = 4;
constexpr int kQStride = 32 + 8;  // bf16 elements of a row of 32 queries, rows apart in the banks

struct TrainTile {
  uint16_t h1[kH][kQStride], dz2[kH][kQStride], dz1[kH][kQStride], x[kXStride][kQStride];
};
struct TrainSums {
  float part[kPartial];
  float upper[3][kH];  // b1, b2, w3: the sums of lanes 16..31 (lanes 0..15 in part)
};

// a tile's LDS contents pass between the lanes of the one wave that owns it
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// rows k0..k0+7 of column q from an operand's eight elements
__device__ __forceinline__ void scatter_operand(uint16_t (*rows)[kQStride], int k0, int q, bf16x8 v) {
  const uint4 u = __builtin_bit_cast(uint4, v);
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    rows[k0 + 2 * j][q] = (uint16_t)w[j];
    rows[k0 + 2 * j + 1][q] = (uint16_t)(w[j] >> 16);
  }
}

// the sum over the lane's row of 16
__device__ __forceinline__ float row_sum16(float v) {
  v += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x128, 0xF, 0xF, true));  // row_ror:8
  v += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x124, 0xF, 0xF, true));  // row_ror:4
  v += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x122, 0xF, 0xF, true));  // row_ror:2
  v += __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), 0x121, 0xF, 0xF, true));  // row_ror:1
  return v;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(64 * kTrainWaves, 1) void k_mlp_train(const MlpPacked* P, const float* x,
                                                                   const float* t_target, int64_t n,
                                                                   float* partials) {
  __shared__ __align__(16) RowConsts c;
  __shared__ __align__(16) uint16_t w2t[kH][kH + 8];
  __shared__ __align__(16) union {
    TrainTile tile[kTrainWaves];
    TrainSums sums[kTrainWaves];
  } lds;
  for (int i = threadIdx.x; i < kH * kH / 8; i += blockDim.x)
    *reinterpret_cast<bf16x8*>(&w2t[i / 8][8 * (i % 8)]) = global_bf16x8(&P->w2t[i / 8][8 * (i % 8)]);
  stage_consts(c, P);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, half = lane >> 5;
  const RegWeights w = load_weights(P, lane);
  const float b3 = P->b3;
  TrainTile& tl = lds.tile[wave];
  f32x16 gw2[2][2] = {};
  f32x4 gw1[4] = {};  // 16x16x32 products: dW1 rows 16 a .. 16 a + 15, columns l % 16
  f32x16 gb1[2] = {}, gb2[2] = {}, gw3[2] = {};
  float gb3 = 0.f, loss = 0.f;
  const float inv_n = 1.f / (float)n;
  const int64_t step = (int64_t)gridDim.x * kTrainWaves * 32;
  RowSource in(x, n);
  float v[kIn];
  int64_t q0 = ((int64_t)blockIdx.x * kTrainWaves + wave) * 32;
  in.start(q0 + lr, step);
  if (q0 < n) in.load(v);
  for (; q0 < n; q0 += step) {
    const int64_t q = q0 + lr;
    const bool valid = q < n;
    const float m0 = valid ? x[q * 8 + 7] : 0.f, target = valid ? t_target[q] : 0.f;
    const bf16x8 xo = input_operand(v, lane);
    if (q0 + step < n) {
      in.advance();
      in.load(v);
    }
    float s[16], t[16];
    f32x16 d1[2], d2[2], h2[2];
    bf16x8 op[4];
    asm volatile("" ::: "memory");  // the constants are read anew, not kept in registers
    mlp_tile<2>(w, c, xo, lane, s, d1, d2, op, h2);
    wave_lds_fence();  // the products of the tile before have read theirs
    scatter_operand(tl.x, 8 * half, lr, xo);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) scatter_operand(tl.h1, 16 * kt + 8 * half, lr, op[kt]);
#pragma unroll
    for (int r = 0; r < 16; ++r) {  // both halves end with all of the query's terms
      t[r] = s[r];
      swap_halves(s[r], t[r]);
    }
    // loss and d loss / d out of the query
    const float f = sigmoid(sum_terms(b3, s, t));
    const float tp = __expf(-m0 * f);
    const float diff = valid ? tp - target : 0.f;
    const float dout = valid ? 2.f * diff * inv_n * (-m0 * tp) * f * (1.f - f) : 0.f;
    if (half == 0) {
      loss += diff * diff;
      gb3 += dout;
    }
    // dZ2; dw3, db2; dH1^T = W2^T dZ2^T
    f32x16 dz[2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 q4 = *reinterpret_cast<const float4*>(&c.w3[32 * m + 8 * g + 4 * half]);
        const float qq[4] = {q4.x, q4.y, q4.z, q4.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = 4 * g + j;
          gw3[m][r] = fmaf(h2[m][r], dout, gw3[m][r]);
          dz[m][r] = dout * qq[j] * d2[m][r];
          gb2[m][r] += dz[m][r];
        }
      }
    column_operand(dz, op);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) scatter_operand(tl.dz2, 16 * kt + 8 * half, lr, op[kt]);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      dz[m] = f32x16{};
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) dz[m] = mfma(lds_bf16x8(&w2t[32 * m + lr][16 * kt + 8 * half]), op[kt], dz[m]);
    }
    // dZ1; db1
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        dz[m][r] *= d1[m][r];
        gb1[m][r] += dz[m][r];
      }
    column_operand(dz, op);
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) scatter_operand(tl.dz1, 16 * kt + 8 * half, lr, op[kt]);
    wave_lds_fence();
    // dW2 += dZ2^T H1, dW1 (unfolded over the 16 input slots) += dZ1^T X
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      bf16x8 a[2], b[2];
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        a[m] = lds_bf16x8(&tl.dz2[32 * m + lr][16 * kt + 8 * half]);
        b[m] = lds_bf16x8(&tl.h1[32 * m + lr][16 * kt + 8 * half]);
      }
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int k = 0; k < 2; ++k) gw2[m][k] = mfma(a[m], b[k], gw2[m][k]);
    }
    const bf16x8 xb = lds_bf16x8(&tl.x[lane & 15][8 * (lane >> 4)]);
#pragma unroll
    for (int m = 0; m < 4; ++m)
      gw1[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          lds_bf16x8(&tl.dz1[16 * m + (lane & 15)][8 * (lane >> 4)]), xb, gw1[m], 0, 0, 0);
  }
  __syncthreads();  // the tiles' storage becomes the waves' sums
  TrainSums& out = lds.sums[wave];
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) out.part[Q_W1 + (16 * m + 4 * (lane >> 4) + r) * kXStride + (lane & 15)] = gw1[m][r];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = 32 * m + c_row(r, lane);
#pragma unroll
      for (int k = 0; k < 2; ++k) out.part[Q_W2 + row * kH + 32 * k + lr] = gw2[m][k][r];
      const float s1 = row_sum16(gb1[m][r]), s2 = row_sum16(gb2[m][r]), s3 = row_sum16(gw3[m][r]);
      if (lr == 0) {
        out.part[Q_B1 + row] = s1;
        out.part[Q_B2 + row] = s2;
        out.part[Q_W3 + row] = s3;
      } else if (lr == 16) {
        out.upper[0][row] = s1;
        out.upper[1][row] = s2;
        out.upper[2][row] = s3;
      }
    }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    gb3 += __shfl_xor(gb3, m, 64);
    loss += __shfl_xor(loss, m, 64);
  }
  if (lane == 0) {
    out.part[Q_B3] = gb3;
    out.part[Q_LOSS] = loss;
#pragma unroll
    for (int i = Q_LOSS + 1; i < kPartial; ++i) out.part[i] = 0.f;
  }
  __syncthreads();
  float* row = partials + (size_t)blockIdx.x * kPartial;
  for (int i = threadIdx.x; i < kPartial; i += blockDim.x) {
    const int u = i >= Q_B1 && i < Q_W2 ? i - Q_B1 : (i >= Q_B2 && i < Q_B3 ? kH + i - Q_B2 : -1);
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < kTrainWaves; ++k) {
      sum += lds.sums[k].part[i];
      if (u >= 0) sum += (&lds.sums[k].upper[0][0])[u];
    }
    row[i] = sum;
  }
}

// Sum the blocks' partials in a fixed order and fold dW1's hi/lo halves. One
// block per 64 partial columns (a multiple of dW1's row of 16, so its halves
// meet in one block), its 16 waves taking every 16th partial row with eight
// rows' loads in flight, added up in wave order. Bound by latency: the 256
// rows (5.4 MB) of a batch of 65536 in 4.4 us; 1024 rows took 9.6 us so, and 448 us
// with one thread per parameter walking them one load at a time.
constexpr int kReduceWaves = 16;

__global__ __launch_bounds__(64 * kReduceWaves) void k_mlp_reduce(const float* partials, int n_rows, int64_t n,
                                                                  float* grad, float* loss) {
  __shared__ float red[kReduceWaves][64];
  const int col = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int qi = blockIdx.x * 64 + col;
  float s = 0.f;
  if (qi < kPartial) {
    const float* src = partials + qi;
    int w = grp;
    for (; w + 7 * kReduceWaves < n_rows; w += 8 * kReduceWaves) {
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = src[(size_t)(w + k * kReduceWaves) * kPartial];
#pragma unroll
      for (int k = 0; k < 8; ++k) s += v[k];
    }
    for (; w < n_rows; w += kReduceWaves) s += src[(size_t)w * kPartial];
  }
  red[grp][col] = s;
  __syncthreads();
  if (grp != 0) return;
  float t = 0.f;
#pragma unroll
  for (int g = 0; g < kReduceWaves; ++g) t += red[g][col];
  if (qi < Q_B1) {
    // dW1 [64][16]: columns 0..6 and 7..13 of a row are the two halves of its 7
    const float lo = __shfl(t, (col + kIn) & 63, 64);
    const int nn = qi / kXStride, k = qi % kXStride;
    if (k < kIn) grad[O_W1 + nn * kIn + k] = t + lo;
  } else if (qi < Q_LOSS) {
    grad[O_B1 + qi - Q_B1] = t;  // the remaining parameters lie in the same order
  } else if (qi == Q_LOSS && loss) {
    *loss = t / (float)n;
  }
}
static_assert(Q_B1 % 64 == 0 && O_B1 - Q_B1 == O_B3 - Q_B3, "the partials' columns after dW1 follow theta's order");

__global__ __launch_bounds__(256) void k_adam(float* th, float* m, float* v, const float* g, int64_t count, float lr,
                                              float b1, float b2, float eps, float c1, float c2) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  float gi = g[i];
  float mi = b1 * m[i] + (1.f - b1) * gi;
  float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---------------------------------------------------------------------------
int mlp_param_count() { return kParams; }
size_t mlp_packed_bytes() { return sizeof(MlpPacked); }

static int mlp_grid(int64_t n, int waves) {
  int64_t chunks = (n + 63) / 64;
  int64_t blocks = (chunks + waves - 1) / waves;
  return (int)(blocks < 1024 ? (blocks < 1 ? 1 : blocks) : 1024);
}

// one block a compute unit at most: its weight gradients fill the registers
static int train_grid(int64_t n) {
  const int64_t blocks = (n + 32 * kTrainWaves - 1) / (32 * kTrainWaves);
  return (int)(blocks < 256 ? (blocks < 1 ? 1 : blocks) : 256);
}

size_t mlp_workspace_bytes(int64_t n) { return (size_t)train_grid(n) * kPartial * sizeof(float); }

hipError_t launch_mlp_pack(const float* theta, void* packed, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_pack, dim3(kH * kH / 256), dim3(256), 0, s, theta, (MlpPacked*)packed);
  return hipGetLastError();
}

hipError_t launch_mlp_forward_gather(const void* packed, const float* pixfeat, int64_t n_pix, const int* q_pix,
                                     const float* q_z, const unsigned long long* q_count, int64_t q_cap, float* f,
                                     hipStream_t s) {
  if (q_cap <= 0 || n_pix <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_forward_gather, dim3(mlp_grid(q_cap, 4)), dim3(256), 0, s, (const MlpPacked*)packed,
                     pixfeat, q_pix, q_z, q_count, q_cap, n_pix, f);
  return hipGetLastError();
}

hipError_t launch_mlp_table(const void* packed, const float* pixfeat, int64_t n_pix, int n_nodes, float* tab,
                            hipStream_t s) {
  if (n_pix <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_table, dim3(mlp_grid(n_pix * n_nodes, 4)), dim3(256), 0, s, (const MlpPacked*)packed,
                     pixfeat, n_pix, n_nodes, tab);
  return hipGetLastError();
}

hipError_t launch_mlp_input_grad_gather(const void* packed, const float* pixfeat, int64_t n_pix, const int* q_pix,
                                        const float* q_z, const unsigned long long* q_count, int64_t q_cap,
                                        float* out_g, hipStream_t s) {
  if (q_cap <= 0 || n_pix <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_input_grad_gather, dim3(mlp_grid(q_cap, 4)), dim3(256), 0, s, (const MlpPacked*)packed,
                     pixfeat, q_pix, q_z, q_count, q_cap, n_pix, out_g);
  return hipGetLastError();
}

hipError_t launch_mlp_forward(const void* packed, const float* x, int64_t n, float* f, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mlp_forward, dim3(mlp_grid(n, 4)), dim3(256), 0, s, (const MlpPacked*)packed, x, n, f);
  return hipGetLastError();
}

hipError_t launch_mlp_loss_grad(const void* packed, const float* x, const float* t, int64_t n, float* grad,
                                float* loss, float* ws, hipStream_t s) {
  const int grid = train_grid(n);
  hipLaunchKernelGGL(k_mlp_train, dim3(grid), dim3(64 * kTrainWaves), 0, s, (const MlpPacked*)packed, x, t, n, ws);
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kPartial + 63) / 64), dim3(64 * kReduceWaves), 0, s, ws,
                     grid, n, grad, loss);
  return hipGetLastError();
}

hipError_t launch_adam(float* th, float* m, float* v, const float* g, int64_t count, int step, float lr, float b1,
                       float b2, float eps, hipStream_t s) {
  float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, th, m, v, g, count, lr, b1, b2,
                     eps, c1, c2);
  return hipGetLastError();
}

}  // namespace mb
