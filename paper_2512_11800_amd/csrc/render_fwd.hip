// Forward render: one workgroup per 16x16 tile (one thread per pixel, each
// wave an 8x8 quadrant). The tile's Gaussian list is streamed through LDS in
// batches of 256 records, three times:
//   pass 0  the pixel's moment variable (mean and spread of its depth mass),
//   pass 1  warped power moments, Eqs. 10-12, summed in double (Moment pass),
//   setup   Cholesky of the Hankel matrix, kept as L^-1 (Sec. 3.2),
//   pass 2  per-Gaussian quadrature, Eq. 7 / App. B, against the bounds
//           (Quadrature pass), accumulating sum q_i (r, g, b, 1),
//   epilogue  Eq. 15 rescaling (Rescale pass).
// Pass 0 tests coverage and stores, per list entry and wave, the 64-bit mask
// of covered pixels; the later passes (and the backward kernel) walk the
// masks instead. Here the masks are transposed into one word of entries per
// pixel: every lane walks its own pixel's entries (see word_rounds, walk_pairs).
// The kernel is bound by VALU issue. With the pairs of all three passes queued in
// (entry, pixel) order and their results summed by owner loops through LDS it
// took 1.17 ms (K = 4), 1.97 ms (K = 6) in the case step_1080p of perf/cases.py (500k
// Gaussians, 1920x1080), against 0.91 and 1.71 ms: what went is the queueing, the
// broadcasts and the owner loops. Every pixel's sums keep their order and every pair its arithmetic: the
// image, the saved state and the moments are the same to the last bit (a
// degenerate pixel's gradients magnify a changed bit by four decades), except where
// a Gaussian reaches over the near bound: the edges moved there round in another order.
//
// Variants (MODE):
//   kModePlain    the path above;
//   kModeHarvest  the same, also writing a seeded pseudo-random subset of its
//                 queries as training samples of the learned surrogate
//                 (features, query, m_0 and the transmittance of the bounds);
//   kModeEmit     passes 0-1, then the surrogate's query list in place of the
//                 bound evaluation; k_render_consume completes the quadrature
//                 from the surrogate's outputs.
#include "render_common.h"
#include "trig.h"

namespace mb {

// Surrogate features of a pixel: the moments of its normalised measure in
// standardised form (mean 0, variance 1 in the moment variable), passed
// through asinh, and the map (y - mu) / sig of the moment variable onto the
// standardised one. The moment bounds are covariant under increasing affine
// maps of the variable, so F at a query depends on these alone.
__device__ __forceinline__ void surrogate_features(const double* acc, float* feat, float& mu, float& sig) {
  double b[7];
  b[0] = 1.0;
#pragma unroll
  for (int k = 1; k <= 6; ++k) b[k] = acc[k] / acc[0];
  const double m = b[1];
  const double var = b[2] - m * m;
  const double s = var > 0.0 ? sqrt(var) : 1.0;
  const double is = 1.0 / s;
  double c[7];  // central moments E[(y - m)^k]
  c[0] = 1.0;
#pragma unroll
  for (int k = 1; k <= 6; ++k) {
    // sum_j C(k, j) b_j (-m)^(k - j), with binomials built by the recurrence
    double acc_k = 0.0, binom = 1.0, pw = 1.0;
#pragma unroll
    for (int j = k; j >= 0; --j) {
      acc_k += binom * b[j] * pw;
      binom = binom * (double)j / (double)(k - j + 1);
      pw *= -m;
    }
    c[k] = acc_k;
  }
  double sk = 1.0;
#pragma unroll
  for (int k = 1; k <= 6; ++k) {
    sk *= is;
    feat[k - 1] = (float)asinh(c[k] * sk);
  }
  mu = (float)m;
  sig = (float)s;
}

// 32-bit integer hash for the harvest's sample selection
__device__ __forceinline__ uint32_t mix_hash(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t h = a * 0x9E3779B1u ^ (b + 0x7F4A7C15u) * 0x85EBCA77u ^ (c + 0x165667B1u) * 0xC2B2AE3Du;
  h ^= h >> 16;
  h *= 0x7FEB352Du;
  h ^= h >> 15;
  h *= 0x846CA68Bu;
  h ^= h >> 16;
  return h;
}

constexpr float kMaxZ = 10.f;  // clamp of the standardised query

__device__ __forceinline__ float std_query(float y, float mu, float sig) {
  return fminf(fmaxf((y - mu) / sig, -kMaxZ), kMaxZ);
}

// acc += m with m rounded first, not fused into the product that formed it
__device__ __forceinline__ void add_rounded(double& acc, double m) {
  asm("" : "+v"(m));
  acc += m;
}

// The wide form (WIDE), for frames of few tiles: a block takes one quadrant of a
// tile, and its four waves evaluate the pixels' pairs four at a time, wave w the
// pixel's pairs 4 i + w; after each step every wave adds the four results in list
// order, so that all sums are the ordinary form's to the last bit. LDS holds a step's
// results, V floats a pair, twice, `half` floats apart (a wave may run one step ahead).
// eval(j, v): entry j against this lane's pixel; add(v): its share of the sums.
// In the ordinary form a tile is one block and each quadrant one wave, and few tiles
// leave most of the chip idle. Ordinary -> wide, K = 4, 6 and 8 (three intervals):
//   64 tiles, 128x128, 2000 Gaussians       96 -> 63, 165 -> 98, 314 -> 173 us
//   475 tiles, 397x301, 20000               401 -> 225, 784 -> 417, 1668 -> 917 us
//   1200 tiles, 640x480, 10000              299 -> 249, 609 -> 462, 1286 -> 1102 us
//   1200 tiles, 100000                      1.80 -> 1.55, 3.68 -> 3.27, 8.61 -> 8.31 ms
//   1200 tiles, 200000, most of them split  3.26 -> 3.04, 6.67 -> 6.41, 15.8 -> 16.6 ms
//   1900 tiles, 10000                       337 -> 360, 687 -> 678, 1503 -> 1629 us
//   1900 tiles, 100000                      2.51 -> 2.36, 5.28 -> 5.04, 12.1 -> 13.1 ms
//   3072 tiles, 10000                       422 -> 541, 860 -> 1037, 1870 -> 2516 us
// A split tile is the same work in both forms, with K = 8 at two blocks a compute unit
// instead of three. Beyond 1200 tiles the lanes without a pair in a step cost more than
// the waves bring. Trigonometric K = 4: 216 -> 108 us at 64 tiles, 1.07 -> 0.55 ms at
// 475, 4.60 -> 4.19 ms at 1200 (100000).
template <int V, class Eval, class Add>
__device__ __forceinline__ void wide_rounds(float* buf, int half, const uint64_t* masks, int b, int nb, int quad, int lane,
                                            int wave, bool live, int& step, Eval&& eval, Add&& add) {
  const int nc = n_chunks(nb, -1);
  for (int c = 0; c < nc; ++c) {
    const uint64_t word = transpose_masks(load_masks(masks, b, nb, quad, -1, c, lane), lane);
    uint64_t m = live ? word : 0ull;
    int left = __popcll(m);
    for (int w = 0; w < wave; ++w) m &= m - 1;
    while (__ballot(left > 0) != 0) {  // the same in all four waves
      float* to = buf + (step & 1) * half;
      if (m != 0) {
        float v[V];
        eval(chunk_entry(c, (int)__builtin_ctzll(m), -1), v);
#pragma unroll
        for (int k = 0; k < V; ++k) to[(wave * V + k) * 64 + lane] = v[k];
#pragma unroll
        for (int w = 0; w < 4; ++w) m &= m - 1;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < 4; ++w)
        if (w < left) {
          float v[V];
#pragma unroll
          for (int k = 0; k < V; ++k) v[k] = to[(w * V + k) * 64 + lane];
          add(v);
        }
      left -= 4;
      ++step;
    }
  }
}

template <int K, int NQ, int MODE, bool WIDE = false>
__global__
// waves per SIMD: five for K = 4 (0.91 ms against 0.92 ms with four, in the case above),
// four for K = 6 (1.71 against 1.85 ms with three) and for the trigonometric K = 4
// (0.54 against 0.59 ms with three, 200k Gaussians, 1280x720; fused operations issue
// slower at an odd number of waves), three beyond. The same with five intervals, where
// they spill 16 (K = 4), 11 (K = 6) and 22 registers (trigonometric) and the fewer
// waves none: K = 4 1.15 ms either way in the case above, 0.21 against 0.19 ms with
// four (100k Gaussians, 1003x757); K = 6 2.39 against 2.48 and 0.41 against 0.40 ms with
// three; trigonometric K = 4 0.71 against 0.77 ms with three (1280x720). K = 8 with
// five intervals: 0.85 ms with three, 0.90 with four (1003x757), 5.5 and 5.4 ms in the
// case above. The wide form: as many as its LDS and registers allow without spills.
__launch_bounds__(256, WIDE ? (MODE == kModeTrig ? 2 : (K == 4 ? 4 : (K == 6 ? 3 : 2))) : (K == 4 ? (MODE == kModeTrig ? 4 : 5) : (K == 6 && MODE == kModePlain ? 4 : 3)))
void k_render_fwd(RenderArgs a, CamSet cams) {
  constexpr int NH = K / 2;
  __shared__ Stage st;
  __shared__ long long s_base;
  __shared__ int s_scan[4];
  const int tiles_per_cam = a.tiles_x * a.tiles_y;
  const int n_keys = tiles_per_cam * a.n_cams;
  static_assert(!WIDE || MODE == kModePlain || MODE == kModeTrig, "the wide form is that of the whole render");
  WideWork bw;
  if constexpr (WIDE) {
    bw = wide_work(a, n_keys);
  } else {
    const BlockWork b = block_work(a);
    bw = {b.key, b.quad, b.quad >= 0};
  }
  const int key = bw.key;
  if (key >= n_keys) return;
  const int ci = key / tiles_per_cam;
  const int tile = key - ci * tiles_per_cam;
  const int ty = tile / a.tiles_x, tx = tile - ty * a.tiles_x;
  const CamConst& c = cams.c[ci];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int2 rg = a.ranges[key];
  // the wave's 8x8 pixel block; in a split block all four waves share one
  // and each takes every fourth list entry (own4)
  const bool split = bw.split;
  const bool wide = WIDE && !split;
  const int quad = WIDE || split ? bw.quad : wave;
  const int own4 = split ? wave : -1;
  const bool writer = wide ? wave == 0 : own4 <= 0;  // of the pixel's sums, which all of its waves hold
  const int px = tx * kTile + (quad & 1) * 8 + (lane & 7);
  const int py = ty * kTile + (quad >> 1) * 8 + (lane >> 3);
  const bool inside = px < c.width && py < c.height;
  const float u = (float)px + 0.5f, v = (float)py + 0.5f;
  const float fi = (float)(px - tx * kTile), fj = (float)(py - ty * kTile);  // offset inside the tile
  const float rx = (u - c.cx) / c.fx, ry = (v - c.cy) / c.fy;
  const float lam = sqrtf(1.f + rx * rx + ry * ry);
  const float tn = c.tn;
  const size_t pix = ((size_t)ci * c.height + (inside ? py : 0)) * c.width + (inside ? px : 0);

  constexpr bool kTrig = MODE == kModeTrig;
  constexpr bool kDblMom = K >= 8 || kTrig;  // moments per pair in double
  // a step's results in the wide form: four pairs of a pixel's moments, or of its sums of pass 2
  constexpr int kWideHalf = 4 * 64 * (kDblMom ? 2 * (K + 1) : (K + 1 > 5 ? K + 1 : 5));
  __shared__ WaveQueue wq[4];
  __shared__ float band[kBlock];  // per staged entry: the coverage test's rounding band (cover_setup)
  // results of the queued pairs of pass 2: q (r, g, b, 1), consistency penalty
  __shared__ __align__(16) float wres[WIDE ? 1 : 4][WIDE ? 2 * kWideHalf : 5 * 64];
  WaveQueue& q = wq[wave];
  float* res = &wres[0][0] + wave * 5 * 64;
  float* wbuf = &wres[0][0];  // the wide form's
  const int x0 = tx * kTile + (quad & 1) * 8, y0 = ty * kTile + (quad >> 1) * 8;
  // partial per-pixel sums of a split block's four waves, combined in wave
  // order through the (then idle) staging buffer; every wave ends with the
  // same totals
  float* xch = reinterpret_cast<float*>(&st);
  int step = 0;
  // this lane's pixel against staged entry j
  auto ray_own = [&](int j) __attribute__((always_inline)) {
    return ray_params(st, j, u - st.f[0][j].x, v - st.f[0][j].y, lam);
  };
  // a list of one batch stays staged from pass 0 on
  const bool staged = rg.y - rg.x <= kBlock;

  // ---- pass 0: coverage masks and the pixel's moment variable --------------
  // weighted depth statistics of the covering Gaussians (weight omega Sigma):
  // sums of w, w mu and w (mu^2 + Sigma^2) in double (weights can be denormal
  // floats; the variance is a difference of these sums)
  double sw = 0.0, swm = 0.0, swq = 0.0;
  int n_cov = 0;
  {
    const uint64_t inside_mask = __ballot(inside);
    for (int b = rg.x; b < rg.y; b += kBlock) {
      int nb = min(kBlock, rg.y - b);
      __syncthreads();
      load_batch(st, a.rec, a.sorted_rec, b, nb);
      // each thread reads back the record it staged itself
      if (tid < nb) band[tid] = cover_setup(st, tid, tx * kTile, ty * kTile);
      __syncthreads();
      const int nc = n_chunks(nb, own4);
      for (int ch = wide ? wave : 0; ch < nc; ch += wide ? 4 : 1) {
        const int jl = chunk_entry(ch, lane, own4);
        const bool mine = jl < nb;
        const int jr = mine ? jl : 0;
        float near;
        uint64_t mask = cover_entry(st, jr, quad, near);
        uint64_t amb = __ballot(mine && near < band[jr]);
        while (amb) {
          const int l = __builtin_ctzll(amb);
          amb &= amb - 1;
          const int j = chunk_entry(ch, l, own4);
          const uint64_t exact = __ballot(covers(st, band[j], a.rectd, a.sorted_rec, b, j, fi, fj, u, v));
          mask = lane == l ? exact : mask;
        }
        mask = mine ? mask & inside_mask : 0ull;
        if (mine) a.masks[(size_t)(b + jl) * 4 + quad] = mask;
        if (wide) continue;
        const uint64_t word = transpose_masks(mask, lane);
        n_cov += __popcll(word);
        word_rounds(word, ch, own4, [&](int j) __attribute__((always_inline)) {
          const RayG g = ray_own(j);
          const double wgt = (double)(g.omega * g.sig), mu = (double)g.mu, sg = (double)g.sig;
          sw += wgt;
          swm = fma(wgt, mu, swm);
          swq = fma(wgt, fma(mu, mu, sg * sg), swq);
        });
      }
      if (wide) {
        __syncthreads();  // all of the batch's masks
        wide_rounds<3>(
            wbuf, kWideHalf, a.masks, b, nb, quad, lane, wave, true, step,
            [&](int j, float* v) __attribute__((always_inline)) {
              const RayG g = ray_own(j);
              v[0] = g.omega * g.sig;
              v[1] = g.mu;
              v[2] = g.sig;
            },
            [&](const float* v) __attribute__((always_inline)) {
              const double wgt = (double)v[0], mu = (double)v[1], sg = (double)v[2];
              ++n_cov;
              sw += wgt;
              swm = fma(wgt, mu, swm);
              swq = fma(wgt, fma(mu, mu, sg * sg), swq);
            });
      }
    }
  }
  if (split) {
    // add the four waves' sums in wave order
    double* xd = reinterpret_cast<double*>(&st);
    __syncthreads();
    xd[(wave * 4 + 0) * 64 + lane] = sw;
    xd[(wave * 4 + 1) * 64 + lane] = swm;
    xd[(wave * 4 + 2) * 64 + lane] = swq;
    xd[(wave * 4 + 3) * 64 + lane] = (double)n_cov;
    __syncthreads();
    sw = swm = swq = 0.0;
    n_cov = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      sw += xd[(w * 4 + 0) * 64 + lane];
      swm += xd[(w * 4 + 1) * 64 + lane];
      swq += xd[(w * 4 + 2) * 64 + lane];
      n_cov += (int)xd[(w * 4 + 3) * 64 + lane];
    }
  }
  float mean = 0.f, var = 0.f;
  if (sw > 0.0) {
    const double md = swm / sw;
    mean = (float)md;
    var = (float)fmax(swq / sw - md * md, 0.0);
  }
  float tc = fmaxf(mean, tn);
  float sd = var > 0.f ? sqrtf(var) : 1.f;
  {
    float qq = 1.f + 0.8f * tc, xn = 1.f + 0.8f * tn;
    float gp = 1.2f * xn * sqrtf(xn) / (qq * qq * sqrtf(qq));  // g_hat'(tc)
    sd = fmaxf(sd * gp, 1e-30f);
  }
  const PixelBasis pb = make_basis(tc, sd, tn);

  // ---- pass 1: moments ------------------------------------------------------
  double acc[K + 1];
#pragma unroll
  for (int k = 0; k <= K; ++k) acc[k] = 0.0;
  {
    for (int b = rg.x; b < rg.y; b += kBlock) {
      int nb = min(kBlock, rg.y - b);
      if (!staged) {
        __syncthreads();
        load_batch_covered(st, a.rec, a.sorted_rec, a.masks, bw.quad, b, nb);
        __syncthreads();
      }
      if (wide) {
        if constexpr (kDblMom) {
          wide_rounds<2 * (K + 1)>(
              wbuf, kWideHalf, a.masks, b, nb, quad, lane, wave, true, step,
              [&](int j, float* v) __attribute__((always_inline)) {
                double m[K + 1];
                if constexpr (kTrig)
                  particle_trig_moments_d<NH>(ray_own(j), tn, m);
                else
                  particle_moments_d<K>(ray_own(j), pb, tn, m);
#pragma unroll
                for (int k = 0; k <= K; ++k) {
                  v[2 * k] = __int_as_float(__double2loint(m[k]));
                  v[2 * k + 1] = __int_as_float(__double2hiint(m[k]));
                }
              },
              [&](const float* v) __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k <= K; ++k)
                  acc[k] += __hiloint2double(__float_as_int(v[2 * k + 1]), __float_as_int(v[2 * k]));
              });
        } else {
          wide_rounds<K + 1>(
              wbuf, kWideHalf, a.masks, b, nb, quad, lane, wave, true, step,
              [&](int j, float* v) __attribute__((always_inline)) { particle_moments<K>(ray_own(j), pb, tn, v); },
              [&](const float* v) __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k <= K; ++k) acc[k] += (double)v[k];
              });
        }
        continue;
      }
      for_each_own_entry(a.masks, b, nb, quad, own4, lane, true, [&](int j) __attribute__((always_inline)) {
        const RayG g = ray_own(j);
        if constexpr (kTrig) {
          double m[K + 1];
          particle_trig_moments_d<NH>(g, tn, m);
#pragma unroll
          for (int k = 0; k <= K; ++k) add_rounded(acc[k], m[k]);
        } else if constexpr (kDblMom) {
          double m[K + 1];
          particle_moments_d<K>(g, pb, tn, m);
#pragma unroll
          for (int k = 0; k <= K; ++k) add_rounded(acc[k], m[k]);
        } else {
          float m[K + 1];
          particle_moments<K>(g, pb, tn, m);
#pragma unroll
          for (int k = 0; k <= K; ++k) acc[k] += (double)m[k];
        }
      });
    }
  }

  if (split) {
    double* xd = reinterpret_cast<double*>(&st);
    __syncthreads();
#pragma unroll
    for (int k = 0; k <= K; ++k) xd[(wave * (K + 1) + k) * 64 + lane] = acc[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k <= K; ++k) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < 4; ++w) t += xd[(w * (K + 1) + k) * 64 + lane];
      acc[k] = t;
    }
  }
  // the backward pass starts from these sums (one column per moment)
  if (inside && writer) {
#pragma unroll
    for (int k = 0; k <= K; ++k) a.pix_mom[(size_t)k * a.n_pix + pix] = acc[k];
  }

  // ---- per-pixel setup ------------------------------------------------------
  const float m0 = (float)acc[0];
  // a pixel whose optical depth is below kMinDepth is empty: its radiance
  // (about m0 times a colour) is negligible, and its moment vector is too close
  // to the float32 underflow range to define a measure
  const bool live = acc[0] > kMinDepth;
  LInv<NH> L = {};
  Orth<MODE == kModeTabPlain ? NH : 2> orth = {};
  TrigLInv<kTrig ? NH : 1> TL;
  bool fallback = false;
  if constexpr (kTrig) {
    if (live) fallback = trig_factor<NH>(acc, TL) != 0.0;
  } else if constexpr (MODE != kModeEmit && MODE != kModeTabSur) {
    if (live) {
      double bn[K + 1], bmix[K + 1];
      bn[0] = 1.0;
#pragma unroll
      for (int k = 1; k <= K; ++k) bn[k] = acc[k] / acc[0];
      if constexpr (MODE == kModeTabPlain)
        fallback = hankel_orth<NH>(bn, orth) != 0.0;
      else
        fallback = hankel_factor<NH>(bn, L, bmix) != 0.0;
    }
  }

  float feat[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float smu = 0.f, ssig = 1.f;
  if constexpr (MODE == kModeHarvest || MODE == kModeEmit || MODE == kModeTabSur) {
    static_assert(K == 6, "the surrogate takes six moments");
    if (live) surrogate_features(acc, feat, smu, ssig);
  }

  // ---- tabulated schedule: the pixel's record (and the bounds' table) -------
  if constexpr (MODE == kModeTabPlain || MODE == kModeTabSur) {
    if constexpr (MODE == kModeTabPlain) {
      if (live) {
        const double mb = acc[1] / acc[0];
        const double var = acc[2] / acc[0] - mb * mb;
        smu = (float)mb;
        ssig = (float)(var > 0.0 ? sqrt(var) : 1.0);
      }
    }
    if (inside && own4 <= 0) {
      float* pf = a.pixfeat + pix * kPixFeat;
#pragma unroll
      for (int k = 0; k < 6; ++k) pf[k] = feat[k];
      pf[6] = live ? m0 : 0.f;
      pf[7] = tc;
      pf[8] = sd;
      // covering count, as -(count + 1) where the bounds' measure was degenerate
      pf[9] = fallback ? -(float)(n_cov + 1) : (float)n_cov;
      pf[10] = smu;
      pf[11] = ssig;
      if constexpr (MODE == kModeTabPlain) {
        // the moment bounds at the nodes y_g = mean + sd z_g
        const float dz = 2.f * kTabZ / (float)(a.tab_nodes - 1);
        float* tp = a.tab + pix * a.tab_nodes;
        for (int g = 0; live && g < a.tab_nodes; ++g)  // an empty pixel's table is never read
          tp[g] = orth_F<NH>(orth, fmaf(orth.l2, smu + ssig * (-kTabZ + dz * (float)g), orth.l1), a.beta);
      }
    }
    return;
  }

  // ---- surrogate query list: this tile's range, pixel by pixel --------------
  long long qbase = -1;
  if constexpr (MODE == kModeEmit) {
    const int nq = (inside && live) ? n_cov * NQ : 0;
    int inc = nq;  // inclusive scan over the wave, then over the 4 waves
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      int t = __shfl_up(inc, d, 64);
      if (lane >= d) inc += t;
    }
    if (lane == 63) s_scan[wave] = inc;
    __syncthreads();
    int off = inc - nq, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      off += w < wave ? s_scan[w] : 0;
      tot += s_scan[w];
    }
    if (tid == 0) s_base = tot > 0 ? (long long)atomicAdd(a.q_count, (unsigned long long)tot) : 0;
    __syncthreads();
    const long long base = s_base;
    // past the capacity the tile's pixels get no queries; the counter still
    // reports the full request so the caller can size the list and retry.
    // A reservation that straddles the capacity fills its part below it with
    // a harmless query (pixel 0), so every slot below min(count, capacity)
    // names a pixel of the image.
    if (base + tot <= a.q_cap) {
      if (inside && live) qbase = base + off;
    } else {
      for (long long i = base + tid; i < a.q_cap; i += kBlock) {
        a.q_z[i] = 0.f;
        a.q_pix[i] = 0;
      }
    }
    if (inside) {
      float* pf = a.pixfeat + pix * kPixFeat;
#pragma unroll
      for (int k = 0; k < 6; ++k) pf[k] = feat[k];
      pf[6] = m0;
      pf[7] = tc;
      pf[8] = sd;
      pf[9] = (float)n_cov;
      a.pix_qbase[pix] = qbase;
    }
  }

  // ---- pass 2: quadrature (or the surrogate's query list) -------------------
  float sr = 0.f, sg = 0.f, sb = 0.f, so = 0.f, spen = 0.f;
  const bool want_pen = a.penalty != nullptr;
  if constexpr (MODE == kModeEmit) {
    int i_pair = 0;
    for (int b = rg.x; b < rg.y; b += kBlock) {
      int nb = min(kBlock, rg.y - b);
      __syncthreads();
      load_batch(st, a.rec, a.sorted_rec, b, nb);
      __syncthreads();
      // the pairs of the coverage masks pass 0 stored (their count is n_cov)
      for_each_own_entry(a.masks, b, nb, quad, own4, lane, inside && live, [&](int j) __attribute__((always_inline)) {
        const RayG g = ray_own(j);
        QEdges<NQ> e;
        quad_edges<NQ>(g, pb, tn, a, e);
        if (qbase >= 0) {
#pragma unroll
          for (int k = 0; k < NQ; ++k) {
            const long long qi = qbase + (long long)i_pair * NQ + k;
            a.q_z[qi] = std_query(e.y[k], smu, ssig);
            a.q_pix[qi] = (int)pix;
          }
        }
        ++i_pair;
      });
    }
    return;
  } else {
    float4* cb = reinterpret_cast<float4*>(res);  // [64]
    float* cpen = res + 256;                       // [64] consistency penalty
    for (int b = rg.x; b < rg.y; b += kBlock) {
      int nb = min(kBlock, rg.y - b);
      if (!staged) {
        __syncthreads();
        load_batch_covered(st, a.rec, a.sorted_rec, a.masks, bw.quad, b, nb);
        __syncthreads();
      }
      if (wide) {
        wide_rounds<5>(
            wbuf, kWideHalf, a.masks, b, nb, quad, lane, wave, inside && live, step,
            [&](int j, float* v) __attribute__((always_inline)) {
              const RayG g = ray_own(j);
              QEdges<NQ> e;
              float qv;
              if constexpr (kTrig)
                qv = particle_quadrature_trig<NH, NQ>(g, TL, m0, tn, a, e);
              else
                qv = particle_quadrature<NH, NQ>(g, pb, L, m0, tn, a, e);
              const float4 f5 = st.f[5][j];
              v[0] = qv * f5.y;
              v[1] = qv * f5.z;
              v[2] = qv * f5.w;
              v[3] = qv;
              v[4] = want_pen ? pair_penalty<NQ>(g, tn, e, a) : 0.f;
            },
            [&](const float* v) __attribute__((always_inline)) {
              sr += v[0];
              sg += v[1];
              sb += v[2];
              so += v[3];
              spen += v[4];
            });
        continue;
      }
      auto eval = [&](bool direct, bool on, int j, int p, uint64_t own) __attribute__((always_inline)) {
        // the pixel's values: the lane's own, or those of pixel lane p
        PixelBasis pp = pb;
        LInv<NH> Lp = L;
        TrigLInv<kTrig ? NH : 1> TLp = TL;
        float m0p = m0, lamp = lam, up = u, vp = v;
        float featp[6], smup = smu, ssigp = ssig;
#pragma unroll
        for (int f = 0; f < 6; ++f) featp[f] = feat[f];
        if (!direct) {
          m0p = from_lane(m0, p);
          if constexpr (kTrig) {
#pragma unroll
            for (int i = 0; i < (NH + 1) * (NH + 2) / 2; ++i) {
              TLp.re[i] = from_lane(TL.re[i], p);
              TLp.im[i] = from_lane(TL.im[i], p);
            }
          } else {
            pp.tc = from_lane(pb.tc, p);
            pp.p = from_lane(pb.p, p);
            pp.p15 = from_lane(pb.p15, p);
            pp.amp = from_lane(pb.amp, p);
#pragma unroll
            for (int i = 0; i < (NH + 1) * (NH + 2) / 2; ++i) Lp.l[i] = from_lane(L.l[i], p);
          }
          lamp = from_lane(lam, p);
          up = (float)(x0 + (p & 7)) + 0.5f;
          vp = (float)(y0 + (p >> 3)) + 0.5f;
          if constexpr (MODE == kModeHarvest) {
#pragma unroll
            for (int f = 0; f < 6; ++f) featp[f] = from_lane(feat[f], p);
            smup = from_lane(smu, p);
            ssigp = from_lane(ssig, p);
          }
        }
        float4 c4 = make_float4(0.f, 0.f, 0.f, 0.f);
        float pen = 0.f;
        if (on) {
          const RayG g = ray_params(st, j, up - st.f[0][j].x, vp - st.f[0][j].y, lamp);
          QEdges<NQ> e;
          float qv;
          if constexpr (kTrig) {
            qv = particle_quadrature_trig<NH, NQ>(g, TLp, m0p, tn, a, e);
          } else {
            qv = particle_quadrature<NH, NQ>(g, pp, Lp, m0p, tn, a, e);
          }
          if constexpr (MODE == kModeHarvest) {
            const uint32_t rid = (uint32_t)a.sorted_rec[b + j];
            const size_t pixp = ((size_t)ci * c.height + (y0 + (p >> 3))) * c.width + (x0 + (p & 7));
#pragma unroll
            for (int k = 0; k < NQ; ++k) {
              const uint32_t h = mix_hash(a.seed, (uint32_t)pixp, rid * NQ + k);
              if ((float)(h >> 8) * (1.f / 16777216.f) < a.harvest_rate) {
                const int slot = atomicAdd(a.harvest_count, 1);
                if (slot < a.harvest_cap) {
                  float* o = a.harvest + (size_t)slot * kHarvestStride;
#pragma unroll
                  for (int f = 0; f < 6; ++f) o[f] = featp[f];
                  o[6] = std_query(e.y[k], smup, ssigp);
                  o[7] = m0p;
                  o[8] = expf(-e.tau[k]);
                  o[9] = __uint_as_float(h);
                  o[10] = __int_as_float((int)pixp);
                  o[11] = __int_as_float((int)(rid * NQ + k));
                }
              }
            }
          }
          const float4 f5 = st.f[5][j];
          c4 = make_float4(qv * f5.y, qv * f5.z, qv * f5.w, qv);
          if (want_pen) pen = pair_penalty<NQ>(g, tn, e, a);
        }
        if (direct) {
          // zero in the lanes without a pair; rounded, not fused into the sums
          // (as the queued results are)
          asm("" : "+v"(c4.x), "+v"(c4.y), "+v"(c4.z), "+v"(pen));
          sr += c4.x;
          sg += c4.y;
          sb += c4.z;
          so += c4.w;
          spen += pen;
        } else {
          cb[lane] = c4;
          if (want_pen) cpen[lane] = pen;
          __builtin_amdgcn_wave_barrier();
          while (own) {
            const int i = __builtin_ctzll(own);
            own &= own - 1;
            const float4 o4 = cb[i];
            sr += o4.x;
            sg += o4.y;
            sb += o4.z;
            so += o4.w;
            if (want_pen) spen += cpen[i];
          }
          __builtin_amdgcn_wave_barrier();
        }
      };
      // Trigonometric K = 6 iterates for a zero, and a wave waits for its slowest lane.
      // The pixels of one entry need much the same steps, those of a round's many
      // entries do not: walked by pixel words the kernel took 1.45 ms (three
      // intervals) and 2.01 ms (five), entry by entry it takes 1.36 and 1.88 ms
      // (200k Gaussians, 1280x720); 0.85 -> 0.79 ms at 100k, 1003x757.
      if constexpr (kTrig && K == 6) {
        walk_entries<true>(
            q, a.masks, b, nb, quad, own4, lane, __ballot(inside && live),
            [&](const Window& w) __attribute__((always_inline)) {
              const bool on = lane < w.n;
              const int it = on ? (int)q.item[w.base + lane] : lane;
              eval(false, on, on ? it >> 6 : 0, it & 63, w.own);
            },
            [](int) {});
      } else {
        walk_pairs(q, a.masks, b, nb, quad, own4, lane, inside && live, eval);
      }
    }
  }

  if (split) {
    __syncthreads();
    xch[(wave * 5 + 0) * 64 + lane] = sr;
    xch[(wave * 5 + 1) * 64 + lane] = sg;
    xch[(wave * 5 + 2) * 64 + lane] = sb;
    xch[(wave * 5 + 3) * 64 + lane] = so;
    xch[(wave * 5 + 4) * 64 + lane] = spen;
    __syncthreads();
    sr = sg = sb = so = spen = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      sr += xch[(w * 5 + 0) * 64 + lane];
      sg += xch[(w * 5 + 1) * 64 + lane];
      sb += xch[(w * 5 + 2) * 64 + lane];
      so += xch[(w * 5 + 3) * 64 + lane];
      spen += xch[(w * 5 + 4) * 64 + lane];
    }
    if (wave != 0) return;
  }
  if (!writer) return;

  // ---- epilogue: Eq. 15 ------------------------------------------------------
  if (!inside) return;
  float alpha = -expm1f(-m0);
  float tr = expf(-m0);
  float inv_o = 1.f / fmaxf(a.eps, so);
  float* out = a.image + pix * 3;
  out[0] = alpha * sr * inv_o + tr * c.bg[0];
  out[1] = alpha * sg * inv_o + tr * c.bg[1];
  out[2] = alpha * sb * inv_o + tr * c.bg[2];
  float4* sv = reinterpret_cast<float4*>(a.saved + pix * MB_SAVED_FLOATS_PER_PIXEL);
  sv[0] = make_float4(sr, sg, sb, so);
  if (want_pen) a.penalty[pix] = spen;
  // covering count; stored as -(count + 1) when the pixel's measure was
  // degenerate (mixed with a normal, or the identity factor; see hankel_factor)
  sv[1] = make_float4(tc, sd, m0, fallback ? -(float)(n_cov + 1) : (float)n_cov);
}

// Second half of the surrogate forward: Eq. 7 with the optical depth m_0 F
// from the surrogate's outputs for the queries the emit pass listed, in the
// same pair order (query index = pixel base + pair * NQ + edge).
template <int NQ>
__global__ __launch_bounds__(256) void k_render_consume(RenderArgs a, CamSet cams) {
  __shared__ Stage st;
  const int tiles_per_cam = a.tiles_x * a.tiles_y;
  const int n_keys = tiles_per_cam * a.n_cams;
  const int key = block_work(a).key;  // the surrogate path splits no tile
  if (key >= n_keys) return;
  const int ci = key / tiles_per_cam;
  const int tile = key - ci * tiles_per_cam;
  const int ty = tile / a.tiles_x, tx = tile - ty * a.tiles_x;
  const CamConst& c = cams.c[ci];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int px = tx * kTile + (wave & 1) * 8 + (lane & 7);
  const int py = ty * kTile + (wave >> 1) * 8 + (lane >> 3);
  const bool inside = px < c.width && py < c.height;
  const float u = (float)px + 0.5f, v = (float)py + 0.5f;
  const float rx = (u - c.cx) / c.fx, ry = (v - c.cy) / c.fy;
  const float lam = sqrtf(1.f + rx * rx + ry * ry);
  const float tn = c.tn;
  const int2 rg = a.ranges[key];
  const size_t pix = ((size_t)ci * c.height + (inside ? py : 0)) * c.width + (inside ? px : 0);
  const float* pf = a.pixfeat + pix * kPixFeat;
  const float m0 = inside ? pf[6] : 0.f;
  const long long qbase = inside ? a.pix_qbase[pix] : -1;
  const bool active = qbase >= 0;
  const PixelBasis pb = make_basis(inside ? pf[7] : tn, inside ? pf[8] : 1.f, tn);
  float sr = 0.f, sg = 0.f, sb = 0.f, so = 0.f;
  int i_pair = 0;
  for (int b = rg.x; b < rg.y; b += kBlock) {
    int nb = min(kBlock, rg.y - b);
    __syncthreads();
    load_batch(st, a.rec, a.sorted_rec, b, nb);
    __syncthreads();
    // the pairs of the forward pass's coverage masks, in the emit pass's order
    for_each_own_entry(a.masks, b, nb, wave, -1, lane, active, [&](int j) __attribute__((always_inline)) {
      const float dx = u - st.f[0][j].x, dy = v - st.f[0][j].y;
      RayG g = ray_params(st, j, dx, dy, lam);
      QEdges<NQ> e;
      quad_edges<NQ>(g, pb, tn, a, e);
      const float* fq = a.q_f + qbase + (long long)i_pair * NQ;
      // the bounds the surrogate stands for grow with depth: its optical
      // depth along the edges is made non-decreasing (running maximum; a
      // later edge takes over only when strictly larger)
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        const float tk = m0 * fq[k];
        e.tau[k] = (k == 0 || tk > e.tau[k > 0 ? k - 1 : 0]) ? tk : e.tau[k > 0 ? k - 1 : 0];
      }
      float q = quad_sum<NQ>(g, tn, e);
      float4 f5 = st.f[5][j];
      sr += q * f5.y;
      sg += q * f5.z;
      sb += q * f5.w;
      so += q;
      ++i_pair;
    });
  }
  if (!inside) return;
  float alpha = -expm1f(-m0);
  float tr = expf(-m0);
  float inv_o = 1.f / fmaxf(a.eps, so);
  float* out = a.image + pix * 3;
  out[0] = alpha * sr * inv_o + tr * c.bg[0];
  out[1] = alpha * sg * inv_o + tr * c.bg[1];
  out[2] = alpha * sb * inv_o + tr * c.bg[2];
  float4* sv = reinterpret_cast<float4*>(a.saved + pix * MB_SAVED_FLOATS_PER_PIXEL);
  sv[0] = make_float4(sr, sg, sb, so);
  sv[1] = make_float4(pf[7], pf[8], m0, pf[9]);
}

// Second half of the tabulated schedule: Eq. 7 and Eq. 15 with the optical
// depth at every edge interpolated linearly in the pixel's table at the
// edge's standardised query (clamped to the table's ends), made
// non-decreasing along the edges (a running maximum; the surrogate's table
// need not grow, the bounds' table does).
template <int NQ>
__global__ __launch_bounds__(256) void k_render_consume_tab(RenderArgs a, CamSet cams) {
  __shared__ Stage st;
  __shared__ WaveQueue wq[4];
  __shared__ __align__(16) float4 wres[4][64];
  const int tiles_per_cam = a.tiles_x * a.tiles_y;
  const int n_keys = tiles_per_cam * a.n_cams;
  const int key = block_work(a).key;  // the tabulated schedule splits no tile
  if (key >= n_keys) return;
  const int ci = key / tiles_per_cam;
  const int tile = key - ci * tiles_per_cam;
  const int ty = tile / a.tiles_x, tx = tile - ty * a.tiles_x;
  const CamConst& c = cams.c[ci];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int x0 = tx * kTile + (wave & 1) * 8, y0 = ty * kTile + (wave >> 1) * 8;
  const int px = x0 + (lane & 7), py = y0 + (lane >> 3);
  const bool inside = px < c.width && py < c.height;
  const float u = (float)px + 0.5f, v = (float)py + 0.5f;
  const float rx = (u - c.cx) / c.fx, ry = (v - c.cy) / c.fy;
  const float lam = sqrtf(1.f + rx * rx + ry * ry);
  const float tn = c.tn;
  const int2 rg = a.ranges[key];
  const size_t pix = ((size_t)ci * c.height + (inside ? py : 0)) * c.width + (inside ? px : 0);
  const float* pf = a.pixfeat + pix * kPixFeat;
  const float m0 = inside ? pf[6] : 0.f;
  const bool active = inside && m0 > 0.f;
  const PixelBasis pb = make_basis(inside ? pf[7] : tn, inside ? pf[8] : 1.f, tn);
  const float smu = inside ? pf[10] : 0.f, isig = inside ? 1.f / pf[11] : 1.f;
  const float ucoef = (float)(a.tab_nodes - 1) / (2.f * kTabZ);
  WaveQueue& q = wq[wave];
  float4* res = wres[wave];
  float sr = 0.f, sg = 0.f, sb = 0.f, so = 0.f;
  for (int b = rg.x; b < rg.y; b += kBlock) {
    int nb = min(kBlock, rg.y - b);
    __syncthreads();
    load_batch_covered(st, a.rec, a.sorted_rec, a.masks, -1, b, nb);
    __syncthreads();
    // as the quadrature pass of k_render_fwd
    walk_pairs(q, a.masks, b, nb, wave, -1, lane, active,
               [&](bool direct, bool on, int j, int p, uint64_t own) __attribute__((always_inline)) {
      PixelBasis pp = pb;
      float m0p = m0, lamp = lam, smup = smu, isigp = isig;
      if (!direct) {
        pp.tc = from_lane(pb.tc, p);
        pp.p = from_lane(pb.p, p);
        pp.p15 = from_lane(pb.p15, p);
        pp.amp = from_lane(pb.amp, p);
        m0p = from_lane(m0, p);
        lamp = from_lane(lam, p);
        smup = from_lane(smu, p);
        isigp = from_lane(isig, p);
      }
      float4 c4 = make_float4(0.f, 0.f, 0.f, 0.f);
      if (on) {
        const int ppx = x0 + (p & 7), ppy = y0 + (p >> 3);
        const float dx = (float)ppx + 0.5f - st.f[0][j].x;
        const float dy = (float)ppy + 0.5f - st.f[0][j].y;
        RayG g = ray_params(st, j, dx, dy, lamp);
        QEdges<NQ> e;
        quad_edges<NQ>(g, pp, tn, a, e);
        const float* tp = a.tab + (((size_t)ci * c.height + ppy) * c.width + ppx) * a.tab_nodes;
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
          const float z = fminf(fmaxf((e.y[k] - smup) * isigp, -kTabZ), kTabZ);
          const float uu = (z + kTabZ) * ucoef;
          const int i0 = min((int)uu, a.tab_nodes - 2);
          const float fr = uu - (float)i0;
          const float f = fmaf(fr, tp[i0 + 1] - tp[i0], tp[i0]);
          const float tk = m0p * f;
          e.tau[k] = (k == 0 || tk > e.tau[k > 0 ? k - 1 : 0]) ? tk : e.tau[k > 0 ? k - 1 : 0];
        }
        const float qv = quad_sum<NQ>(g, tn, e);
        const float4 f5 = st.f[5][j];
        c4 = make_float4(qv * f5.y, qv * f5.z, qv * f5.w, qv);
      }
      if (direct) {
        sr += c4.x;
        sg += c4.y;
        sb += c4.z;
        so += c4.w;
      } else {
        res[lane] = c4;
        __builtin_amdgcn_wave_barrier();
        while (own) {
          const int i = __builtin_ctzll(own);
          own &= own - 1;
          const float4 o4 = res[i];
          sr += o4.x;
          sg += o4.y;
          sb += o4.z;
          so += o4.w;
        }
        __builtin_amdgcn_wave_barrier();
      }
    });
  }
  if (!inside) return;
  float alpha = -expm1f(-m0);
  float tr = expf(-m0);
  float inv_o = 1.f / fmaxf(a.eps, so);
  float* out = a.image + pix * 3;
  out[0] = alpha * sr * inv_o + tr * c.bg[0];
  out[1] = alpha * sg * inv_o + tr * c.bg[1];
  out[2] = alpha * sb * inv_o + tr * c.bg[2];
  float4* sv = reinterpret_cast<float4*>(a.saved + pix * MB_SAVED_FLOATS_PER_PIXEL);
  sv[0] = make_float4(sr, sg, sb, so);
  sv[1] = make_float4(pf[7], pf[8], m0, pf[9]);
}

hipError_t launch_render_consume_tab(const RenderArgs& a, const CamSet& cams, int n_intervals, hipStream_t s) {
  int n_keys = a.tiles_x * a.tiles_y * a.n_cams;
  dim3 grid(render_blocks(n_keys)), block(kBlock);
  if (n_intervals == 3)
    hipLaunchKernelGGL(k_render_consume_tab<4>, grid, block, 0, s, a, cams);
  else if (n_intervals == 5)
    hipLaunchKernelGGL(k_render_consume_tab<6>, grid, block, 0, s, a, cams);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_render_forward(const RenderArgs& a, const CamSet& cams, int n_moments, int n_intervals,
                                 hipStream_t s, int mode) {
  int n_keys = a.tiles_x * a.tiles_y * a.n_cams;
  dim3 grid(render_blocks(n_keys)), block(kBlock);
#define MB_LAUNCH_WIDE(KK, NN, MM)                                                                           \
  if (wide && n_moments == KK && n_intervals == NN && mode == MM) {                                          \
    hipLaunchKernelGGL((k_render_fwd<KK, NN + 1, MM, true>), dim3(4 * n_keys), block, 0, s, a, cams);        \
    return hipGetLastError();                                                                                \
  }
  // (not the trigonometric K = 6, whose sums follow the compiler's choice of fused
  // operations in the last bit)
  const bool wide = n_keys <= kWideTiles;
  MB_LAUNCH_WIDE(4, 3, kModePlain)
  MB_LAUNCH_WIDE(6, 3, kModePlain)
  MB_LAUNCH_WIDE(4, 5, kModePlain)
  MB_LAUNCH_WIDE(6, 5, kModePlain)
  MB_LAUNCH_WIDE(8, 3, kModePlain)
  MB_LAUNCH_WIDE(8, 5, kModePlain)
  MB_LAUNCH_WIDE(4, 3, kModeTrig)
  MB_LAUNCH_WIDE(4, 5, kModeTrig)
#undef MB_LAUNCH_WIDE
#define MB_LAUNCH(KK, NN, MM)                                                       \
  if (n_moments == KK && n_intervals == NN && mode == MM) {                         \
    hipLaunchKernelGGL((k_render_fwd<KK, NN + 1, MM>), grid, block, 0, s, a, cams); \
    return hipGetLastError();                                                       \
  }
  MB_LAUNCH(4, 3, kModePlain)
  MB_LAUNCH(6, 3, kModePlain)
  MB_LAUNCH(4, 5, kModePlain)
  MB_LAUNCH(6, 5, kModePlain)
  MB_LAUNCH(8, 3, kModePlain)
  MB_LAUNCH(8, 5, kModePlain)
  MB_LAUNCH(6, 3, kModeHarvest)
  MB_LAUNCH(6, 5, kModeHarvest)
  MB_LAUNCH(6, 3, kModeEmit)
  MB_LAUNCH(6, 5, kModeEmit)
  MB_LAUNCH(4, 3, kModeTrig)
  MB_LAUNCH(4, 5, kModeTrig)
  MB_LAUNCH(6, 3, kModeTrig)
  MB_LAUNCH(6, 5, kModeTrig)
  MB_LAUNCH(4, 3, kModeTabPlain)
  MB_LAUNCH(6, 3, kModeTabPlain)
  MB_LAUNCH(4, 5, kModeTabPlain)
  MB_LAUNCH(6, 5, kModeTabPlain)
  MB_LAUNCH(6, 3, kModeTabSur)
  MB_LAUNCH(6, 5, kModeTabSur)
#undef MB_LAUNCH
  return hipErrorInvalidValue;
}

hipError_t launch_render_consume(const RenderArgs& a, const CamSet& cams, int n_intervals, hipStream_t s) {
  int n_keys = a.tiles_x * a.tiles_y * a.n_cams;
  dim3 grid(render_blocks(n_keys)), block(kBlock);
  if (n_intervals == 3)
    hipLaunchKernelGGL(k_render_consume<4>, grid, block, 0, s, a, cams);
  else if (n_intervals == 5)
    hipLaunchKernelGGL(k_render_consume<6>, grid, block, 0, s, a, cams);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace mb
