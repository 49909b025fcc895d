// Backward render: the two-stage adjoint of Sec. 3.3 (Eq. 22, App. D), one
// workgroup per 16x16 tile as in the forward pass.
//   pass 1   the pixel's moment sums, as the forward pass stored them (per
//            pixel; nothing per (pixel, Gaussian) pair is stored);
//   setup    Hankel factor; the derivative of the Eq. 15 rescaling is folded
//            in: a = g (1 - e^-m0) / max(eps, O), b = dL/dO, e0 = dL/dm0;
//   pass 2   Adjoint-Moment stage: dm = e0 e_0 + sum_i (a . c_i + b) dq_i/dm,
//            through the quadrature (Eq. 7) and the adjoint of the moment
//            bounds at every interval edge; the same evaluation also gives
//            the part of the Gradient stage that does not depend on dm,
//            (a . c_i + b) dq_i/dtheta_i for theta = (mu, Sigma, omega) and the
//            colour term, chained to the record coefficients;
//   pass 3   the rest of the Gradient stage, dm . dm_i/dtheta_i.
// Per-pair gradients are summed over the wave's pixels into one slot per
// (list entry, wave) (pass 2 writes it, pass 3 adds to it); a per-Gaussian
// kernel then sums the slots: one reduction, no atomics, deterministic. A
// byte per slot records whether it was written (the stored coverage mask of
// that entry and quadrant is non-empty); the reduction skips the others.
// The passes walk the coverage masks the forward pass stored (walk_entries).
// The kernel is bound by VALU issue: per 64 pairs about 3500 issue cycles of pass 2
// and 1400 of pass 3 beside the queueing. With the queue's state in scalar
// registers, the near bound's selects out of the way and the pixels' values in LDS
// it takes 2.21 -> 1.98 ms (K = 4), 3.74 -> 3.15 ms (K = 6) in the case step_1080p of
// perf/cases.py (500k Gaussians, 1920x1080); the gradients are the same bits
// (trigonometric K = 6: equal but for the last bits of the sums).
#include "render_common.h"
#include "trig.h"

namespace mb {

// Quadrature of one Gaussian with the state its adjoint needs.
template <int NH, int NQ>
struct QuadState {
  float t[NQ], y[NQ], w0[NQ], F[NQ], tau[NQ], T[NQ], sr[NQ], off[NQ];
  float x[NQ][NH];
  bool below[NQ][NH];
  bool cl[NQ];  // the edge lies on the near bound; set where `near`
  bool near;    // wave-uniform: some lane's first edge does (the edges ascend)
  float dt[NQ], ph[NQ], dph[NQ], A[NQ];
  float q;
};

// phi'(x) = (e^-x - phi(x)) / x from d = e^-x and phi: the derivative of
// phi's series (terms up to x^4) for |x| < 1/16, the direct form beyond
__device__ __forceinline__ float dphi_fn(float x, float d, float ph) {
  // coefficients (-1)^k k / (k+1)!, k = 1..5
  float s = 5.f / 720.f;
  s = fmaf(s, -x, 4.f / 120.f);
  s = fmaf(s, -x, 3.f / 24.f);
  s = fmaf(s, -x, 2.f / 6.f);
  s = fmaf(s, -x, 0.5f);
  return fabsf(x) < kPhiSeries ? -s : (d - ph) * fast_rcp(x);
}

// Edges of one Gaussian's quadrature (App. B) and sigma_i there. A wave without an
// edge on the near bound takes the short forms here and below: the selects and
// their masks took 2.06 ms where 2.01 do (K = 4), and with the registers they held
// 3.41 ms where 3.20 do (K = 6, spills), in the case step_1080p.
// FUSED: which operations are fused. The optical depths that the adjoint passes
// through follow the edges' last bits, and a degenerate pixel's gradients magnify
// them; the operations are therefore fixed here and do not follow the code around.
template <int NH, int NQ, bool FUSED>
__device__ __forceinline__ void quad_geom(const RayG& g, const PixelBasis& pb, float tn, const RenderArgs& a,
                                          QuadState<NH, NQ>& s) {
  const float mu = rounded(g.mu), ks = rounded(a.kappa * g.sig);
  const float dtc = FUSED ? fmaf(g.id, g.le, -pb.tc) : mu - pb.tc;
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    s.off[j] = rounded(ks * a.xq[j]);
    s.t[j] = fmaf(ks, a.xq[j], mu);
    s.y[j] = FUSED ? fmaf(ks, a.xq[j], dtc) : dtc + s.off[j];
    s.sr[j] = a.eq[j];
    s.cl[j] = false;
  }
  s.near = __ballot(s.t[0] < tn) != 0;
  if (s.near) {
    const float rn = (tn - g.mu) * fast_rcp(g.sig);  // edges moved onto the near bound
    const float en = exp_neg_half(rn * rn);
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      s.cl[j] = s.t[j] < tn;
      s.y[j] = s.cl[j] ? (tn - pb.tc) : s.y[j];
      s.t[j] = s.cl[j] ? tn : s.t[j];
      s.sr[j] = s.cl[j] ? en : s.sr[j];
    }
  }
#pragma unroll
  for (int j = 0; j < NQ; ++j) s.y[j] = warp_y(pb, s.t[j], s.y[j]);
}

// Given the optical depth s.tau at the edges: the Eq. 7 terms, q, and
// A[j] = dq / dtau_j.
template <int NH, int NQ>
__device__ __forceinline__ void quad_terms(const RayG& g, float tn, QuadState<NH, NQ>& s) {
  if (s.near) {
#pragma unroll
    for (int j = 0; j + 1 < NQ; ++j) {
      const float first = s.t[j + 1] - tn, free = s.off[j + 1] - s.off[j];
      s.dt[j] = s.cl[j + 1] ? 0.f : (s.cl[j] ? first : free);
    }
  } else {
#pragma unroll
    for (int j = 0; j + 1 < NQ; ++j) s.dt[j] = s.off[j + 1] - s.off[j];
  }
  s.T[0] = __expf(-s.tau[0]);
  s.q = 0.f;
#pragma unroll
  for (int j = 0; j < NQ; ++j) s.A[j] = 0.f;
#pragma unroll
  for (int j = 0; j + 1 < NQ; ++j) {
    float dtau = s.tau[j + 1] - s.tau[j];
    const float d = __expf(-dtau);
    s.T[j + 1] = s.T[j] * d;
    s.ph[j] = phi_fn(dtau, d);
    s.dph[j] = dphi_fn(dtau, d, s.ph[j]);
    float tds = s.T[j] * s.dt[j] * g.omega * s.sr[j];
    s.q += tds * s.ph[j];
    // dq/dtau_j and dq/dtau_{j+1} of this interval's term
    s.A[j] -= tds * (s.ph[j] + s.dph[j]);
    s.A[j + 1] += tds * s.dph[j];
  }
}

// dq / d(mu, Sigma, omega) at fixed optical depths
template <int NH, int NQ>
__device__ __forceinline__ void quad_position_grads(const RayG& g, const QuadState<NH, NQ>& s, const RenderArgs& a,
                                                    float& dq0, float& dq1, float& dq2) {
  dq0 = dq1 = dq2 = 0.f;
  if (s.near) {
    const float isg = fast_rcp(g.sig);
#pragma unroll
    for (int e = 0; e + 1 < NQ; ++e) {
      const float cdt = s.T[e] * s.ph[e] * g.omega * s.sr[e];
      const float dmu0 = s.cl[e] ? 0.f : 1.f, dmu1 = s.cl[e + 1] ? 0.f : 1.f;
      const float dsg0 = s.cl[e] ? 0.f : a.kxq[e], dsg1 = s.cl[e + 1] ? 0.f : a.kxq[e + 1];
      dq0 += cdt * (dmu1 - dmu0);
      dq1 += cdt * (dsg1 - dsg0);
      const float cs = s.T[e] * s.dt[e] * s.ph[e];
      if (s.cl[e]) {
        const float r = (s.t[e] - g.mu) * isg;
        const float sj = g.omega * s.sr[e];
        dq0 += cs * sj * r * isg;
        dq1 += cs * sj * r * r * isg;
      }
      dq2 += cs * s.sr[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e + 1 < NQ; ++e) {
      dq1 += s.T[e] * s.ph[e] * g.omega * s.sr[e] * a.dkxq[e];
      dq2 += s.T[e] * s.dt[e] * s.ph[e] * s.sr[e];
    }
  }
}

// adds wgt dtau_dt dt_e / d(mu, Sigma) to (gmu, gsig)
template <int NH, int NQ>
__device__ __forceinline__ void edge_position_grads(const QuadState<NH, NQ>& s, const RenderArgs& a,
                                                    const float* gt, float& gmu, float& gsig) {
  if (s.near) {
#pragma unroll
    for (int e = 0; e < NQ; ++e) {
      gmu += gt[e] * (s.cl[e] ? 0.f : 1.f);
      gsig += gt[e] * (s.cl[e] ? 0.f : a.kxq[e]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < NQ; ++e) {
      gmu += gt[e];
      gsig += gt[e] * a.kxq[e];
    }
  }
}

template <int NH, int NQ>
__device__ __forceinline__ void quad_state(const RayG& g, const PixelBasis& pb, const LInv<NH>& L, float m0,
                                           float tn, const RenderArgs& a, QuadState<NH, NQ>& s) {
  quad_geom<NH, NQ, (NH > 2)>(g, pb, tn, a, s);
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    s.F[j] = canon_at<NH>(L, s.y[j], a.beta, s.x[j], s.below[j], s.w0[j]);
    s.tau[j] = m0 * s.F[j];
  }
  quad_terms<NH, NQ>(g, tn, s);
}

// The same for the trigonometric moments (the forward pass's
// particle_quadrature_trig): the edge at depth t queries the angle
// psi = (2 pi - theta) g_hat(t) (kept in s.y), the optical depth is a running
// maximum along the edges, and src[e] names the edge whose query supplied
// edge e's value (the last edge at or before e that raised it).
template <int NH, int NQ>
__device__ __forceinline__ void trig_quad_state(const RayG& g, const TrigLInv<NH>& L, float m0, float tn,
                                                const RenderArgs& a, QuadState<NH, NQ>& s, TrigCanon<NH>* tc,
                                                int* src) {
  cfl start = {__builtin_nanf(""), 0.f};  // the first edge starts from its query point
  s.near = __ballot(g.mu + a.kappa * g.sig * a.xq[0] < tn) != 0;
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    s.off[j] = a.kappa * g.sig * a.xq[j];
    const float t = g.mu + s.off[j];
    s.cl[j] = t < tn;
    s.t[j] = s.cl[j] ? tn : t;
    s.y[j] = kTrigSpan * warp_abs(s.t[j], tn);
    const float r = (s.t[j] - g.mu) * fast_rcp(g.sig);
    s.sr[j] = s.cl[j] ? exp_neg_half(r * r) : a.eq[j];
    s.F[j] = trig_canon<NH>(L, s.y[j], a.beta, tc[j], &start);
    const float tj = m0 * s.F[j];
    const bool up = j == 0 || tj > s.tau[j > 0 ? j - 1 : 0];
    s.tau[j] = up ? tj : s.tau[j > 0 ? j - 1 : 0];
    src[j] = up ? j : src[j > 0 ? j - 1 : 0];
  }
  quad_terms<NH, NQ>(g, tn, s);
}

// Double-precision dual number (one tangent) for the Jacobian of the
// surrogate's inputs with respect to the pixel's moments.
struct DualD {
  double v, d;
  __device__ DualD(double a = 0.0, double b = 0.0) : v(a), d(b) {}
};
__device__ __forceinline__ DualD operator+(DualD a, DualD b) { return DualD(a.v + b.v, a.d + b.d); }
__device__ __forceinline__ DualD operator-(DualD a, DualD b) { return DualD(a.v - b.v, a.d - b.d); }
__device__ __forceinline__ DualD operator*(DualD a, DualD b) { return DualD(a.v * b.v, a.d * b.v + a.v * b.d); }
__device__ __forceinline__ DualD operator/(DualD a, DualD b) {
  double r = a.v / b.v;
  return DualD(r, (a.d - r * b.d) / b.v);
}

// Surrogate inputs as functions of the pixel's moments m_0..m_6, as in the
// forward pass: asinh of the standardised moments 1..6 of b = m / m_0, and
// the standardisation (mean mu, standard deviation sig) of the moment variable.
__device__ __forceinline__ void feat_from_moments(const DualD* m, DualD* feat, DualD& mu, DualD& sig) {
  DualD b[7];
  b[0] = DualD(1.0);
#pragma unroll
  for (int k = 1; k <= 6; ++k) b[k] = m[k] / m[0];
  mu = b[1];
  DualD var = b[2] - mu * mu;
  if (var.v > 0.0) {
    const double sq = sqrt(var.v);
    sig = DualD(sq, 0.5 * var.d / sq);
  } else {
    sig = DualD(1.0);
  }
  const DualD is = DualD(1.0) / sig;
  DualD sk(1.0);
#pragma unroll
  for (int k = 1; k <= 6; ++k) {
    DualD c(0.0), pw(1.0);
    double binom = 1.0;
#pragma unroll
    for (int j = k; j >= 0; --j) {
      c = c + DualD(binom) * b[j] * pw;
      binom = binom * (double)j / (double)(k - j + 1);
      pw = pw * (DualD(0.0) - mu);
    }
    sk = sk * is;
    const DualD u = c * sk;
    feat[k - 1] = DualD(asinh(u.v), u.d / sqrt(1.0 + u.v * u.v));
  }
}

// sum_k dm[k] * d m_k / d(mu, Sigma, omega) for the moments of Eqs. 10-12,
// by reverse-mode differentiation of their recurrence: the moments forward
// (kept in registers), then one adjoint sweep back through the recurrence to
// the shared terms G, G', bn, E, erfc, and from those to (mu, Sigma, omega).
template <int K>
__device__ __forceinline__ void moment_grads(const RayG& g, const PixelBasis& pb, float tn, const float* dmv,
                                             float* out) {
  const float c = kSqrtHalfPi;
  const float mus = fmaxf(g.mu, tn);
  const float ys = warp_y(pb, mus, mus - pb.tc);
  const float Gp = warp_dy(pb, mus);
  const float G = ys + Gp * (g.mu - mus);
  const float q = 1.f + 0.8f * g.mu;
  const float d2 = g.mu > tn ? -3.f * pb.amp * fast_rcp(q * q * q * fast_sqrt(q)) : 0.f;  // y''(mu)
  const float is = fast_rcp(g.sig);
  const float bn = (tn - g.mu) * kInvSqrt2 * is;
  const float E = __expf(-bn * bn);
  const float ec = erfc_fast(bn);
  const float s2 = g.sig * g.sig;
  const float tm = tn - g.mu;
  // primal: m_0, m_1 and m_k = G m_{k-1} + (k-1) v2 m_{k-2} + bnd un^(k-1)
  float m[K + 1], up[K];
  m[0] = g.omega * g.sig * c * ec;
  const float bnd = Gp * g.omega * s2 * E;
  m[1] = G * m[0] + bnd;
  const float un = G + Gp * tm;
  const float v2 = Gp * Gp * s2;
  up[0] = 1.f;
#pragma unroll
  for (int k = 1; k < K; ++k) up[k] = up[k - 1] * un;
#pragma unroll
  for (int k = 2; k <= K; ++k) m[k] = G * m[k - 1] + (float)(k - 1) * v2 * m[k - 2] + bnd * up[k - 1];
  // adjoint sweep
  float a[K + 1];
#pragma unroll
  for (int k = 0; k <= K; ++k) a[k] = dmv[k];
  float gG = 0.f, gv2 = 0.f, gbnd = 0.f, gun = 0.f;
#pragma unroll
  for (int k = K; k >= 2; --k) {
    const float km = (float)(k - 1);
    gG += a[k] * m[k - 1];
    a[k - 1] += a[k] * G;
    gv2 += a[k] * km * m[k - 2];
    a[k - 2] += a[k] * km * v2;
    gbnd += a[k] * up[k - 1];
    gun += a[k] * km * up[k - 2];
  }
  gun *= bnd;
  gG += a[1] * m[0] + gun;
  a[0] += a[1] * G;
  gbnd += a[1];
  float gGp = gun * tm + gv2 * 2.f * Gp * s2 + gbnd * g.omega * s2 * E;
  float gmu = -gun * Gp;
  const float gs2 = gv2 * Gp * Gp + gbnd * Gp * g.omega * E;
  const float gE = gbnd * Gp * g.omega * s2;
  float gom = gbnd * Gp * s2 * E + a[0] * g.sig * c * ec;
  float gsig = a[0] * g.omega * c * ec + gs2 * 2.f * g.sig;
  const float gec = a[0] * g.omega * g.sig * c;
  const float gbn = -2.f * E * (gE * bn + gec * 0.5641895835477563f);  // d erfc/db = -2 E / sqrt(pi)
  gmu += -gbn * kInvSqrt2 * is + gG * Gp + gGp * d2;
  gsig += -gbn * bn * is;
  out[0] = gmu;
  out[1] = gsig;
  out[2] = gom;
}

struct BwdArgs {
  RenderArgs r;
  const float* saved;       // [C,H,W,8]
  const float* grad_image;  // [C,H,W,3]
  const float* grad_penalty;  // [C,H,W] dL/d(consistency penalty), or null
  const int* sorted_k;      // [E] entry index of each sorted list position
  float* partials;          // [E,4,kGradStride]
  uint8_t* used;            // [E,4]: which of an entry's slots this pass writes
};

// (mu, Sigma, omega) gradients of one pair -> gradients of its record
// coefficients (the inverse of ray_params); linear in (gmu, gsig, gom)
__device__ __forceinline__ void chain_record(float gmu, float gsig, float gom, const RayG& g, float lamp, float dx,
                                             float dy, const float4& f2, const float4& f3, const float4& f4,
                                             float* gr) {
  // D, X and the exponential as ray_params evaluated them at this offset
  const float id = g.id, ek = g.ek;
  float gE = gmu * lamp * id;
  float gD = -gmu * g.mu * id - 0.5f * gsig * g.sig * id + 0.5f * gom * g.omega * g.xid * id;
  float gX = -0.5f * gom * g.omega * id;
  gr[G_D0] = gD;
  gr[G_D1X] = 2.f * gD * dx;
  gr[G_D1Y] = 2.f * gD * dy;
  gr[G_D2XX] = gD * dx * dx;
  gr[G_D2XY] = 2.f * gD * dx * dy;
  gr[G_D2YY] = gD * dy * dy;
  gr[G_E0] = gE;
  gr[G_EX] = gE * dx;
  gr[G_EY] = gE * dy;
  gr[G_XXX] = gX * dx * dx;
  gr[G_XXY] = 2.f * gX * dx * dy;
  gr[G_XYY] = gX * dy * dy;
  float gdx = 2.f * gD * (f2.y + f2.w * dx + f3.x * dy) + gE * f3.w + 2.f * gX * (f4.y * dx + f4.z * dy);
  float gdy = 2.f * gD * (f2.z + f3.x * dx + f3.y * dy) + gE * f4.x + 2.f * gX * (f4.z * dx + f4.w * dy);
  gr[G_P0X] = -gdx;
  gr[G_P0Y] = -gdy;
  gr[G_W] = gom * ek;
}

// Staged records without the word that only the coverage test reads.
struct BwdStage {
  float4 r[kRecF4 - 1][kBlock];
  __device__ __forceinline__ const float4& word(int k, int j) const { return r[k == 0 ? 0 : k - 1][j]; }
};
// Stage the batch [b, b + nb) (load_batch_covered for these records). Entries whose masks are empty for the
// pixels of this block (all four quadrants, or the block's one) are never queued,
// and their records are not loaded.
__device__ __forceinline__ void load_batch(BwdStage& st, const float4* rec, const int* sorted_rec,
                                           const uint64_t* masks, int quad, int b, int nb) {
  int tid = threadIdx.x;
  if (tid < nb) {
    const uint64_t* mp = masks + (size_t)(b + tid) * 4;
    bool need;
    if (quad >= 0) {
      need = mp[quad] != 0ull;
    } else {
      const ulonglong2 m01 = reinterpret_cast<const ulonglong2*>(mp)[0];
      const ulonglong2 m23 = reinterpret_cast<const ulonglong2*>(mp)[1];
      need = (m01.x | m01.y | m23.x | m23.y) != 0ull;
    }
    if (need) {
      const float4* src = rec + (size_t)sorted_rec[b + tid] * kRecStride;
      st.r[0][tid] = src[0];
#pragma unroll
      for (int k = 2; k < kRecF4; ++k) st.r[k - 1][tid] = src[k];
    }
  }
}

// positions of the window that end a segment
__device__ __forceinline__ uint64_t segment_heads(const Window& w) {  // positions past the window count as heads
  return w.n < 64 ? w.heads | (~0ull << w.n) : w.heads;
}
__device__ __forceinline__ uint64_t segment_ends(const Window& w) {
  const uint64_t act = w.n < 64 ? (1ull << w.n) - 1 : ~0ull;
  return ((segment_heads(w) >> 1) | (1ull << 63)) & act;
}

// Owner accumulation: calls add(load(i)) for this lane's own queue positions
// i (bits of `own`) in increasing order, two positions per iteration with
// both loads issued before either value is consumed.
template <class Load, class Add>
__device__ __forceinline__ void for_each_own(uint64_t own, Load&& load, Add&& add) {
  while (own) {
    const int i0 = __builtin_ctzll(own);
    own &= own - 1;
    const bool two = own != 0;
    const int i1 = two ? __builtin_ctzll(own) : i0;
    own &= own - 1;
    const auto v0 = load(i0);
    const auto v1 = load(i1);
    add(v0);
    if (two) add(v1);
  }
}

// Segmented inclusive scan over the wave's lanes with DPP moves: four
// shifts inside each 16-lane row (row_shr 1, 2, 4, 8), then the classic
// row_bcast 15 (rows 1 and 3) and row_bcast 31 (rows 2 and 3) steps across
// rows. Each step adds the moved value times a 0/1 mask that keeps the sum
// inside the lane's segment; the masks depend only on the segment layout, so one
// set serves every gradient field. The segment's last lane ends with the segment
// sum.
struct ScanMasks {
  float m[6];
};
__device__ __forceinline__ ScanMasks scan_masks(uint64_t heads) {
  // lane i takes lane i - 2^k of its row where none of the lanes between, nor
  // i itself, begins a segment
  const uint64_t c1 = ~heads & 0xfffefffefffefffeull;
  const uint64_t c2 = c1 & (c1 << 1);
  const uint64_t c4 = c2 & (c2 << 2);
  const uint64_t c8 = c4 & (c4 << 4);
  // rows 1 and 3 take the row before, the upper half lane 31, up to their first head
  const uint32_t r1 = (uint32_t)(heads >> 16) & 0xffffu, r3 = (uint32_t)(heads >> 48);
  const uint32_t hi = (uint32_t)(heads >> 32);
  const uint64_t b15 = ((uint64_t)(((r1 & (0u - r1)) - 1u) & 0xffffu) << 16) |
                       ((uint64_t)(((r3 & (0u - r3)) - 1u) & 0xffffu) << 48);
  const uint64_t b31 = (uint64_t)((hi & (0u - hi)) - 1u) << 32;
  auto one = [](uint64_t m) __attribute__((always_inline)) {
    return __builtin_amdgcn_inverse_ballot_w64(m) ? 1.f : 0.f;
  };
  return {{one(c1), one(c2), one(c4), one(c8), one(b15), one(b31)}};
}
// The scan of the gradient fields in one block of v_fmac_f32 with a DPP
// source (v += (v moved) * mask; the compiler would emit a separate move for
// each), step by step over the fields: all 18, or the 15 record fields when
// the colour fields are zero in every lane (the moment part of the Gradient
// stage). A DPP read of a VGPR written by a VALU instruction needs two wait
// states: within the block every read comes 15 or more instructions after
// the write it depends on, and the s_nop covers the values written just
// before the block.
static_assert(G_COUNT == 18 && G_CR == 15, "the scan blocks are written for 15 record and 3 colour fields");
#define MB_SCAN15(M, CTRL) \
  "v_fmac_f32_dpp %0, %0, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %1, %1, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %2, %2, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %3, %3, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %4, %4, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %5, %5, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %6, %6, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %7, %7, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %8, %8, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %9, %9, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %10, %10, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %11, %11, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %12, %12, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %13, %13, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %14, %14, " M " " CTRL "\n\t"
#define MB_SCAN18(M, CTRL) \
  MB_SCAN15(M, CTRL) \
  "v_fmac_f32_dpp %15, %15, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %16, %16, " M " " CTRL "\n\t" \
  "v_fmac_f32_dpp %17, %17, " M " " CTRL "\n\t"

#define MB_ROW(C) "row_shr:" C " row_mask:0xf bank_mask:0xf bound_ctrl:1"
#define MB_BCAST15 "row_bcast:15 row_mask:0xa bank_mask:0xf bound_ctrl:1"
#define MB_BCAST31 "row_bcast:31 row_mask:0xc bank_mask:0xf bound_ctrl:1"
__device__ __forceinline__ void segment_scan18(float* g, const ScanMasks& s) {
  asm("s_nop 1\n\t"
      MB_SCAN18("%18", MB_ROW("1"))
      MB_SCAN18("%19", MB_ROW("2"))
      MB_SCAN18("%20", MB_ROW("4"))
      MB_SCAN18("%21", MB_ROW("8"))
      MB_SCAN18("%22", MB_BCAST15)
      MB_SCAN18("%23", MB_BCAST31)
      : "+v"(g[0]), "+v"(g[1]), "+v"(g[2]), "+v"(g[3]), "+v"(g[4]), "+v"(g[5]), "+v"(g[6]), "+v"(g[7]),
        "+v"(g[8]), "+v"(g[9]), "+v"(g[10]), "+v"(g[11]), "+v"(g[12]), "+v"(g[13]), "+v"(g[14]),
        "+v"(g[15]), "+v"(g[16]), "+v"(g[17])
      : "v"(s.m[0]), "v"(s.m[1]), "v"(s.m[2]), "v"(s.m[3]), "v"(s.m[4]), "v"(s.m[5]));
}
__device__ __forceinline__ void segment_scan15(float* g, const ScanMasks& s) {
  asm("s_nop 1\n\t"
      MB_SCAN15("%15", MB_ROW("1"))
      MB_SCAN15("%16", MB_ROW("2"))
      MB_SCAN15("%17", MB_ROW("4"))
      MB_SCAN15("%18", MB_ROW("8"))
      MB_SCAN15("%19", MB_BCAST15)
      MB_SCAN15("%20", MB_BCAST31)
      : "+v"(g[0]), "+v"(g[1]), "+v"(g[2]), "+v"(g[3]), "+v"(g[4]), "+v"(g[5]), "+v"(g[6]), "+v"(g[7]),
        "+v"(g[8]), "+v"(g[9]), "+v"(g[10]), "+v"(g[11]), "+v"(g[12]), "+v"(g[13]), "+v"(g[14])
      : "v"(s.m[0]), "v"(s.m[1]), "v"(s.m[2]), "v"(s.m[3]), "v"(s.m[4]), "v"(s.m[5]));
}
#undef MB_BCAST31
#undef MB_BCAST15
#undef MB_ROW
#undef MB_SCAN18
#undef MB_SCAN15

// The slot a segment's last lane adds to (pass 3), loaded before the pass's
// arithmetic so that the load's latency hides behind it.
struct SlotVals {
  float4 s[5];
};
// the lanes that write a slot: the segments' last, but for an entry that goes on
__device__ __forceinline__ uint64_t slot_lanes(const Window& w) {
  return segment_ends(w) & ~(w.continues ? 1ull << 63 : 0ull);
}
__device__ __forceinline__ SlotVals load_slot(const Window& w, int j, const float* partials, const BwdStage& st, int wave) {
  SlotVals v;  // read only by the lanes that load it
  if (__builtin_amdgcn_inverse_ballot_w64(slot_lanes(w))) {
    const float4* slot = reinterpret_cast<const float4*>(partials + ((size_t)__float_as_int(st.word(0, j).z) * 4 + wave) * kGradStride);
#pragma unroll
    for (int f = 0; f < 5; ++f) v.s[f] = slot[f];
  }
  return v;
}

// Per-entry sums of the gradients gr[] of the window's pairs: a segmented scan
// over the lanes sums each entry's pairs and the segment's last lane writes
// (ADD = false) or adds to (ADD = true, with the slot's earlier contents in
// `prev`) the entry's slot. An entry that continues in the next window leaves its
// partial sum there, in `carry`.
template <bool ADD>
__device__ __forceinline__ void scan_window(const Window& w, float* gr) {
  // the moment part (ADD) leaves the colour fields zero: they need no scan
  const ScanMasks sm = scan_masks(segment_heads(w));
  if constexpr (ADD)
    segment_scan15(gr, sm);
  else
    segment_scan18(gr, sm);
}
__device__ __forceinline__ void take_carry(const Window& w, float* gr, int lane, const float* carry) {
  if (w.carried && lane == __builtin_ctzll(segment_ends(w))) {
#pragma unroll
    for (int f = 0; f < G_COUNT; ++f) gr[f] += carry[f];
  }
}
__device__ __forceinline__ void leave_carry(const Window& w, const float* gr, int lane, float* carry) {
  if (w.continues && lane == 63) {
#pragma unroll
    for (int f = 0; f < G_COUNT; ++f) carry[f] = gr[f];
  }
}
template <bool ADD>
__device__ __forceinline__ void write_slots(const Window& w, float* gr, int j, float* partials, const BwdStage& st,
                                            int wave, const SlotVals* prev = nullptr) {
  if (__builtin_amdgcn_inverse_ballot_w64(slot_lanes(w))) {
    float4* slot = reinterpret_cast<float4*>(partials + ((size_t)__float_as_int(st.word(0, j).z) * 4 + wave) * kGradStride);
    if constexpr (ADD) {
      const float* pv = reinterpret_cast<const float*>(prev->s);
#pragma unroll
      for (int f = 0; f < G_COUNT; ++f) gr[f] += pv[f];
    }
    slot[0] = make_float4(gr[0], gr[1], gr[2], gr[3]);
    slot[1] = make_float4(gr[4], gr[5], gr[6], gr[7]);
    slot[2] = make_float4(gr[8], gr[9], gr[10], gr[11]);
    slot[3] = make_float4(gr[12], gr[13], gr[14], gr[15]);
    slot[4] = make_float4(gr[16], gr[17], 0.f, 0.f);
  }
}
template <bool ADD>
__device__ __forceinline__ void reduce_to_slots(const Window& w, float* gr, int j, int lane, float* carry,
                                                float* partials, const BwdStage& st, int wave,
                                                const SlotVals* prev = nullptr) {
  scan_window<ADD>(w, gr);
  take_carry(w, gr, lane, carry);
  leave_carry(w, gr, lane, carry);
  write_slots<ADD>(w, gr, j, partials, st, wave, prev);
  __builtin_amdgcn_wave_barrier();
}

// The wide form, for frames of few tiles: a block takes one quadrant of a tile, and
// the windows of its list go to its four waves in turn. Every wave queues all
// pairs, four windows (a group) at a time, and calls flush(group). The windows are
// the ordinary form's, and all sums keep their order: the gradients are the same bits.
// The ordinary form leaves most of the chip idle there (as in the forward kernel).
// Ordinary -> wide, K = 4, 6 and 8 (three intervals):
//   64 tiles, 128x128, 2000 Gaussians       166 -> 99, 252 -> 125, 412 -> 175 us
//   475 tiles, 397x301, 20000               844 -> 489, 1366 -> 768, 2375 -> 1302 us
//   1200 tiles, 640x480, 10000              651 -> 581, 1063 -> 994, 1828 -> 1544 us
//   1200 tiles, 100000                      4.20 -> 3.59, 6.94 -> 6.99, 13.9 -> 12.0 ms
//   1200 tiles, 200000, most of them split  7.66 -> 6.99, 12.7 -> 14.0, 26.0 -> 24.0 ms
//   1900 tiles, 10000                       760 -> 877, 1250 -> 1519, 2190 -> 2346 us
//   1900 tiles, 100000                      5.92 -> 5.53, 9.93 -> 11.0, 20.1 -> 19.0 ms
//   3072 tiles, 10000                       909 -> 1356, 1523 -> 2372, 2942 -> 3684 us
// Beyond 1200 tiles every variant loses in thin frames. K = 6 loses in dense ones near
// the line already: its ordinary form has three blocks a compute unit, the wide one
// two. With five intervals K = 6 gains there (10.6 -> 9.06 ms at 100000), K = 4 loses
// in thin frames (759 -> 813 us at 10000). Trigonometric K = 4: 296 -> 139 us and 1.59
// -> 0.87 ms at 64 and 475 tiles, 9.11 -> 7.92 ms at 1200 (100000).
struct Group {
  int n, base;         // pairs in the group, its first item in the ring of 512
  uint64_t heads[5];   // of the four windows, entry starts only; [4] the next group's
  uint64_t own[5];
  __device__ __forceinline__ Window window(int k) const {  // k: wave-uniform
    uint64_t h = 0, next = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h = k == i ? heads[i] : h;
      next = k == i ? heads[i + 1] : next;
    }
    Window w;
    w.n = min(max(n - 64 * k, 0), 64);
    w.base = (base + 64 * k) & 511;
    w.carried = w.n > 0 && (h & 1) == 0;
    w.heads = h | 1;
    w.own = 0;
    w.continues = n > 64 * (k + 1) && (next & 1) == 0;
    return w;
  }
};
template <bool OWN, class Flush, class Empty>
__device__ __forceinline__ void walk_groups(uint16_t* ring, const uint64_t* masks, int b, int nb, int quad, int lane,
                                            uint64_t keep, Flush&& flush, Empty&& on_empty) {
  Group g = {};
  for (int j0 = 0; j0 < nb; j0 += 64) {
    const bool in = j0 + lane < nb;
    const uint64_t raw = in ? masks[(size_t)(b + j0 + lane) * 4 + quad] : 0ull;
    const uint64_t mk = raw & keep;
    if (in && mk == 0 && raw != 0) on_empty(j0 + lane);
    uint64_t nz = __ballot(mk != 0);
    while (nz) {
      const int l = __builtin_ctzll(nz);
      nz &= nz - 1;
      const uint32_t mlo = __builtin_amdgcn_readlane((uint32_t)mk, l);
      const uint32_t mhi = __builtin_amdgcn_readlane((uint32_t)(mk >> 32), l);
      const uint64_t m = ((uint64_t)mhi << 32) | mlo;
      const bool cov = __builtin_amdgcn_inverse_ballot_w64(m);
      const int pos = (int)__builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, (uint32_t)g.n));
      if (cov) ring[(g.base + pos) & 511] = (uint16_t)(((j0 + l) << 6) | lane);
      const uint64_t bit = OWN && cov ? 1ull << (pos & 63) : 0ull;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if ((g.n >> 6) == k) {  // the entry's pairs lie in windows k and k + 1
          g.heads[k] |= 1ull << (g.n & 63);
          if constexpr (OWN) {
            g.own[k] |= (pos >> 6) == k ? bit : 0ull;
            g.own[k + 1] |= (pos >> 6) == k ? 0ull : bit;
          }
        }
      g.n += __builtin_popcountll(m);
      if (g.n >= 256) {
        flush(g);
        g.n -= 256;
        g.base ^= 256;
        g.heads[0] = g.heads[4];
        g.own[0] = g.own[4];
#pragma unroll
        for (int k = 1; k < 5; ++k) g.heads[k] = g.own[k] = 0;
      }
    }
  }
  if (g.n > 0) flush(g);
}

// A pixel's values for the lanes that evaluate its pairs: the first S of N in a
// row of LDS, read by 16-byte loads (rows an odd number of 16 bytes apart, spread
// over the banks), the others broadcast from the pixel lane's registers. A shuffle
// a value held 20 more registers through the passes and took 27 LDS instructions
// a window where 5 loads do: 2.01 -> 1.97 ms (K = 4), 3.20 -> 3.15 ms (K = 6) in the
// case step_1080p (3 blocks a compute unit: 2 take 2.54 and 3.93 ms, 4
// with 160 entries staged at a time 1.94 ms but more where lists are long).
template <int S>
struct PixelRows {
  static_assert(S % 8 == 4, "rows of an odd number of 16-byte words");
  float4* r;  // [64][S / 4]
  template <int N>
  __device__ __forceinline__ void put(int lane, const float* v) const {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < S && i < N; i += 4)
      r[lane * (S / 4) + i / 4] = make_float4(v[i], i + 1 < N ? v[i + 1] : 0.f, i + 2 < N ? v[i + 2] : 0.f,
                                              i + 3 < N ? v[i + 3] : 0.f);
    __builtin_amdgcn_wave_barrier();
  }
  // out: pixel lane p's values; mine: this lane's own (all lanes must take part)
  template <int N>
  __device__ __forceinline__ void get(int p, const float* mine, float* out) const {
#pragma unroll
    for (int i = 0; i < S && i < N; i += 4) {
      const float4 v = r[p * (S / 4) + i / 4];
      out[i] = v.x;
      if (i + 1 < N) out[i + 1] = v.y;
      if (i + 2 < N) out[i + 2] = v.z;
      if (i + 3 < N) out[i + 3] = v.w;
    }
#pragma unroll
    for (int i = S; i < N; ++i) out[i] = from_lane(mine[i], p);
  }
};

// A window's results, N floats a pair, in LDS arrays of 16-, 8- and 4-byte elements
template <int N>
struct Results {
  float v[N];
  __device__ __forceinline__ void store(float* res, int i) const {
    constexpr int n4 = N / 4;
#pragma unroll
    for (int k = 0; k < n4; ++k)
      reinterpret_cast<float4*>(res)[64 * k + i] = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
    if constexpr (N & 2) reinterpret_cast<float2*>(res + 256 * n4)[i] = make_float2(v[4 * n4], v[4 * n4 + 1]);
    if constexpr (N & 1) res[64 * (N - 1) + i] = v[N - 1];
  }
  __device__ __forceinline__ void load(const float* res, int i) {
    constexpr int n4 = N / 4;
#pragma unroll
    for (int k = 0; k < n4; ++k) {
      const float4 f = reinterpret_cast<const float4*>(res)[64 * k + i];
      v[4 * k] = f.x;
      v[4 * k + 1] = f.y;
      v[4 * k + 2] = f.z;
      v[4 * k + 3] = f.w;
    }
    if constexpr (N & 2) {
      const float2 f = reinterpret_cast<const float2*>(res + 256 * n4)[i];
      v[4 * n4] = f.x;
      v[4 * n4 + 1] = f.y;
    }
    if constexpr (N & 1) v[N - 1] = res[64 * (N - 1) + i];
  }
};

// MODE 0: the moment bounds of Sec. 3.2 (power moments).
// MODE 1: the backward pass through the learned surrogate (the forward pass
// was mb_render_forward_surrogate): the optical depth at every edge is m_0 F
// with F and dF/d(inputs) from the query list, and the adjoint reaches the
// moments through the surrogate's inputs instead of the moment bounds.
// MODE 2: trigonometric moments (K = 4 or 6: two or three complex moments),
// the adjoint of the reconstruction on the circle (trig_adjoint) and of
// Eq. 14 (trig_moment_grads) in place of the power moments'.
template <int K, int NQ, int MODE>
constexpr int kBwdBlocks = (K <= 6 && NQ == 4 && MODE == 0) ? 3 : 2;  // blocks a compute unit
template <int K, int NQ, int MODE, bool WIDE = false>
__global__ __launch_bounds__(256, (WIDE ? 2 : kBwdBlocks<K, NQ, MODE>)) void k_render_bwd(BwdArgs ba, CamSet cams) {
  constexpr bool SUR = MODE == 1;
  constexpr bool TRIG = MODE == 2;
  static_assert(!WIDE || !SUR, "the wide form is that of the whole adjoint");
  static_assert(!TRIG || K == 4 || K == 6, "the trigonometric path takes two or three complex moments");
  constexpr int NH = K / 2;
  constexpr int NL = (NH + 1) * (NH + 2) / 2;
  constexpr int NRES = SUR ? 9 : K + 1;  // results per queued pair
  // pixel rows: as many values as leave LDS for the blocks the registers allow
  constexpr int S = SUR ? 12 : (kBwdBlocks<K, NQ, MODE> == 3 ? 20 : 28);
  const RenderArgs& a = ba.r;
  __shared__ BwdStage st;
  __shared__ WaveQueue wq[4];
  __shared__ uint16_t ring[WIDE ? 4 : 1][WIDE ? 512 : 1];  // the wide form's queues
  __shared__ uint32_t wrank[4][SUR ? 128 : 1];           // pair ranks (surrogate queries)
  __shared__ __align__(16) float wres[WIDE ? 8 : 4][NRES * 64];  // per queued pair results
  __shared__ float4 prow[WIDE ? 1 : 4][64 * S / 4];      // pixel values (of the block's one quadrant: WIDE)
  __shared__ float carry[WIDE ? 8 : 4][G_COUNT];         // partial slot of an entry split over evaluations
  const int tiles_per_cam = a.tiles_x * a.tiles_y;
  const int n_keys = tiles_per_cam * a.n_cams;
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
  // as in the forward pass: a split block's waves share one quadrant and
  // take every fourth list entry; slots and masks are per (entry, quadrant)
  const bool split = bw.split;
  const bool wide = WIDE && !split;
  const int quad = WIDE || split ? bw.quad : wave;
  const int own4 = split ? wave : -1;
  int par = 0;  // of the wide form's groups
  const int x0 = tx * kTile + (quad & 1) * 8, y0 = ty * kTile + (quad >> 1) * 8;
  const int px = x0 + (lane & 7);
  const int py = y0 + (lane >> 3);
  const bool inside = px < c.width && py < c.height;
  const float u = (float)px + 0.5f, v = (float)py + 0.5f;
  const float rx = (u - c.cx) / c.fx, ry = (v - c.cy) / c.fy;
  const float lam = sqrtf(1.f + rx * rx + ry * ry);
  const float tn = c.tn;
  const int2 rg = a.ranges[key];
  const size_t pix = inside ? ((size_t)ci * c.height + py) * c.width + px : 0;
  WaveQueue& q = wq[wave];
  float* res = wres[wave];
  const PixelRows<S> rows{prow[WIDE ? 0 : wave]};

  float sv[8] = {0.f, 0.f, 0.f, 0.f, tn + 1.f, 1.f, 0.f, 0.f};
  float gi[3] = {0.f, 0.f, 0.f};
  if (inside) {
    const float4* sp = reinterpret_cast<const float4*>(ba.saved + pix * MB_SAVED_FLOATS_PER_PIXEL);
    float4 s0 = sp[0], s1 = sp[1];
    sv[0] = s0.x; sv[1] = s0.y; sv[2] = s0.z; sv[3] = s0.w;
    sv[4] = s1.x; sv[5] = s1.y; sv[6] = s1.z; sv[7] = s1.w;
    gi[0] = ba.grad_image[pix * 3];
    gi[1] = ba.grad_image[pix * 3 + 1];
    gi[2] = ba.grad_image[pix * 3 + 2];
  }
  const bool want_gp = ba.grad_penalty != nullptr;
  const float gpen = (inside && want_gp) ? ba.grad_penalty[pix] : 0.f;
  const PixelBasis pb = make_basis(sv[4], sv[5], tn);

  auto basis_of = [&](int p) __attribute__((always_inline)) {
    PixelBasis r;
    r.tc = from_lane(pb.tc, p);
    r.p = from_lane(pb.p, p);
    r.p15 = from_lane(pb.p15, p);
    r.amp = from_lane(pb.amp, p);
    return r;
  };
  // the pair at the window's position `lane` (entry j, pixel lane p); inactive
  // lanes get p = lane so the cross-lane reads stay uniform
  auto item_of = [&](const Window& w, int& j, int& p) __attribute__((always_inline)) {
    const bool act = lane < w.n;
    const int it = act ? (int)(wide ? ring[wave][w.base + lane] : q.item[w.base + lane]) : lane;
    j = act ? (it >> 6) : 0;
    p = it & 63;
    return act;
  };
  auto offsets_of = [&](int j, int p, float& dx, float& dy) __attribute__((always_inline)) {
    dx = (float)(x0 + (p & 7)) + 0.5f - st.word(0, j).x;
    dy = (float)(y0 + (p >> 3)) + 0.5f - st.word(0, j).y;
  };
  // flags: mark which of the entries' slots this block writes (an entry's
  // slot for a quadrant whose stored mask is empty is neither written nor
  // read: its sum is zero)
  auto stage = [&](int b, int nb, bool flags) __attribute__((always_inline)) {
    __syncthreads();
    load_batch(st, a.rec, a.sorted_rec, a.masks, bw.quad, b, nb);
    if (tid < nb) {
      const int k = ba.sorted_k[b + tid];
      st.r[0][tid].z = __int_as_float(k);  // the entry's index in place of its centre offset (coverage only)
      if (flags) {
        const uint64_t* mp = a.masks + (size_t)(b + tid) * 4;
        if (bw.quad >= 0) {
          ba.used[(size_t)k * 4 + bw.quad] = mp[bw.quad] != 0ull ? 1 : 0;
        } else {
          uchar4 f;
          f.x = mp[0] != 0ull ? 1 : 0;
          f.y = mp[1] != 0ull ? 1 : 0;
          f.z = mp[2] != 0ull ? 1 : 0;
          f.w = mp[3] != 0ull ? 1 : 0;
          reinterpret_cast<uchar4*>(ba.used)[k] = f;
        }
      }
    }
    __syncthreads();
  };

  // ---- the pixel's moment sums, as the forward pass left them --------------
  double acc[K + 1];
#pragma unroll
  for (int k = 0; k <= K; ++k) acc[k] = inside ? a.pix_mom[(size_t)k * a.n_pix + pix] : 0.0;
  const float m0 = (float)acc[0];
  const bool live = acc[0] > kMinDepth;  // as in the forward pass
  LInv<NH> L;
  TrigLInv<TRIG ? NH : 1> TL;
  float bk[K + 1];
  bk[0] = 1.f;
  float mix_eps = 0.f;  // the forward pass's mixture weight (degenerate measures)
  if (live && !SUR) {
    double bn[K + 1], bmix[K + 1];
    bn[0] = 1.0;
#pragma unroll
    for (int k = 1; k <= K; ++k) {
      bn[k] = acc[k] / acc[0];
      bk[k] = (float)bn[k];
    }
    if constexpr (TRIG) {
      mix_eps = (float)trig_factor<NH>(acc, TL);
#pragma unroll
      for (int i = 0; i < NL; ++i) L.l[i] = 0.f;
    } else {
      mix_eps = (float)hankel_factor<NH>(bn, L, bmix);
    }
  } else {
    if constexpr (TRIG) {
#pragma unroll
      for (int i = 0; i < NL; ++i) TL.re[i] = TL.im[i] = 0.f;
    }
#pragma unroll
    for (int k = 1; k <= K; ++k) bk[k] = 0.f;
#pragma unroll
    for (int i = 0; i < NL; ++i) L.l[i] = 0.f;
  }

  // ---- Eq. 15 adjoint, folded into the two stages -------------------------
  const float alpha = -expm1f(-m0);
  const float oc = fmaxf(a.eps, sv[3]);
  float ga[3], gb, e0;
  {
    float gs = gi[0] * sv[0] + gi[1] * sv[1] + gi[2] * sv[2];
    float gbg = gi[0] * c.bg[0] + gi[1] * c.bg[1] + gi[2] * c.bg[2];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) ga[ch] = gi[ch] * alpha / oc;
    gb = sv[3] > a.eps ? -gs * alpha / (sv[3] * sv[3]) : 0.f;
    e0 = expf(-m0) * (gs / oc - gbg);
  }

  const bool active = inside && live;
  const uint64_t active_mask = __ballot(active);
  float* cw = carry[wave];
  // the slot of an entry whose stored mask has pixels, none of which this
  // pass keeps (outside the image, or without density), is written as zero
  auto zero_slot = [&](int j) __attribute__((always_inline)) {
    float4* slot = reinterpret_cast<float4*>(ba.partials + ((size_t)__float_as_int(st.word(0, j).z) * 4 + quad) * kGradStride);
#pragma unroll
    for (int f = 0; f < kGradStride / 4; ++f) slot[f] = make_float4(0.f, 0.f, 0.f, 0.f);
  };

  // ---- pass 2: adjoint moments, and the dm-independent gradients -----------
  float dm[K + 1];
#pragma unroll
  for (int k = 0; k <= K; ++k) dm[k] = 0.f;
  if constexpr (SUR) {
    static_assert(K == 6, "the surrogate takes six moments");
    // the forward pass's standardisation of the moment variable
    float smu = 0.f, ssig = 1.f;
    if (live) {
      const double mb = acc[1] / acc[0];
      const double var = acc[2] / acc[0] - mb * mb;
      smu = (float)mb;
      ssig = (float)(var > 0.0 ? sqrt(var) : 1.0);
    }
    // a pixel the forward pass left without queries (its list overflowed)
    // rendered as empty there and takes no gradient here
    const long long qb = active ? a.pix_qbase[pix] : -1;
    const uint64_t sur_mask = __ballot(qb >= 0);
    float dm0s = 0.f, dmus = 0.f, dsigs = 0.f, dfeat[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    QueueRanks rk{wrank[wave], 0u};
    auto flush = [&](const Window& w) __attribute__((always_inline)) {
      int j, p;
      const bool act = item_of(w, j, p);
      const PixelBasis pp = basis_of(p);
      const float lamp = from_lane(lam, p), m0p = from_lane(m0, p);
      float gap[3] = {from_lane(ga[0], p), from_lane(ga[1], p), from_lane(ga[2], p)};
      const float gbp = from_lane(gb, p);
      const float smup = from_lane(smu, p), ssigp = from_lane(ssig, p);
      const uint32_t qlo = (uint32_t)__shfl((int)(uint32_t)(qb & 0xffffffffll), p, 64);
      const uint32_t qhi = (uint32_t)__shfl((int)(uint32_t)((unsigned long long)qb >> 32), p, 64);
      const long long qbase_p = (long long)(((unsigned long long)qhi << 32) | qlo);
      float gr[G_COUNT];
#pragma unroll
      for (int f = 0; f < G_COUNT; ++f) gr[f] = 0.f;
      if (act) {
        const uint32_t rank = wrank[wave][w.base + lane];
        float dx, dy;
        offsets_of(j, p, dx, dy);
        RayG g = ray_params(st, j, dx, dy, lamp);
        QuadState<NH, NQ> s;
        quad_geom<NH, NQ, false>(g, pp, tn, a, s);
        // F as the forward pass used it; its input gradient beside it
        const long long qi = qbase_p + (long long)rank * NQ;
        const float* qg = a.q_g + qi * 8;
        // the forward pass's running maximum: edge e takes the optical depth
        // of edge src[e] (the last edge at or before e that raised it)
        int src[NQ];
#pragma unroll
        for (int e = 0; e < NQ; ++e) {
          s.F[e] = a.q_f[qi + e];
          const float te = m0p * s.F[e];
          const bool up = e == 0 || te > s.tau[e > 0 ? e - 1 : 0];
          s.tau[e] = up ? te : s.tau[e > 0 ? e - 1 : 0];
          src[e] = up ? e : src[e > 0 ? e - 1 : 0];
        }
        quad_terms<NH, NQ>(g, tn, s);
        float4 f5 = st.word(5, j);
        const float gbar = gap[0] * f5.y + gap[1] * f5.z + gap[2] * f5.w + gbp;
        // dL/dtau gathered onto the edges whose queries supplied it
        float wsrc[NQ];
#pragma unroll
        for (int e = 0; e < NQ; ++e) wsrc[e] = 0.f;
#pragma unroll
        for (int e = 0; e < NQ; ++e) {
#pragma unroll
          for (int e2 = 0; e2 <= e; ++e2) wsrc[e2] += src[e] == e2 ? gbar * s.A[e] : 0.f;
        }
        float c[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float gmu = 0.f, gsig = 0.f, gom = 0.f, gt[NQ];
        const float isg = fast_rcp(ssigp);
#pragma unroll
        for (int e = 0; e < NQ; ++e) {
          const float* ge = qg + e * 8;
          const float wgt = wsrc[e];
          c[0] += wgt * s.F[e];  // tau = m_0 F at fixed inputs
#pragma unroll
          for (int k = 0; k < 6; ++k) c[1 + k] += wgt * m0p * ge[1 + k];
          const float zr = (s.y[e] - smup) / ssigp;
          const float gz = fabsf(zr) < 10.f ? wgt * m0p * ge[7] * isg : 0.f;  // dL/dy at the edge
          c[7] -= gz;       // z = (y - mu) / sig
          c[8] -= gz * zr;
          gt[e] = rounded(gz * warp_dy(pp, s.t[e]));
        }
        edge_position_grads<NH, NQ>(s, a, gt, gmu, gsig);
        float dq0, dq1, dq2;
        quad_position_grads<NH, NQ>(g, s, a, dq0, dq1, dq2);
        gmu += gbar * dq0;
        gsig += gbar * dq1;
        gom += gbar * dq2;
#pragma unroll
        for (int k = 0; k < 9; ++k) res[k * 64 + lane] = c[k];
        chain_record(gmu, gsig, gom, g, lamp, dx, dy, st.word(2, j), st.word(3, j), st.word(4, j), gr);
        gr[G_CR] = s.q * gap[0];
        gr[G_CG] = s.q * gap[1];
        gr[G_CB] = s.q * gap[2];
      }
      __builtin_amdgcn_wave_barrier();
      uint64_t own = w.own;
      while (own) {
        const int i = __builtin_ctzll(own);
        own &= own - 1;
        dm0s += res[i];
#pragma unroll
        for (int k = 0; k < 6; ++k) dfeat[k] += res[(1 + k) * 64 + i];
        dmus += res[7 * 64 + i];
        dsigs += res[8 * 64 + i];
      }
      reduce_to_slots<false>(w, gr, j, lane, cw, ba.partials, st, quad);
    };
    for (int b = rg.x; b < rg.y; b += kBlock) {
      int nb = min(kBlock, rg.y - b);
      stage(b, nb, true);
      walk_entries<true>(q, a.masks, b, nb, quad, own4, lane, sur_mask, flush, zero_slot, &rk);
    }
    // the moment adjoint through the surrogate's inputs (forward-mode Jacobian
    // of the standardised features in double, one moment at a time)
    if (active) {
#pragma unroll 1
      for (int i = 0; i <= 6; ++i) {
        DualD md[7], feat[6], mu, sg;
#pragma unroll
        for (int k = 0; k <= 6; ++k) md[k] = DualD(acc[k], k == i ? 1.0 : 0.0);
        feat_from_moments(md, feat, mu, sg);
        double d = (i == 0 ? (double)dm0s : 0.0) + (double)dmus * mu.d + (double)dsigs * sg.d;
#pragma unroll
        for (int k = 0; k < 6; ++k) d += (double)dfeat[k] * feat[k].d;
        dm[i] = (float)d;
      }
      if (own4 <= 0) dm[0] += e0;
    }
  } else {
  dm[0] = (active && own4 <= 0) ? e0 : 0.f;  // a split block adds e0 once (wave 0)
  // the pixel's values: factor, m_0, lambda, b_1..K, basis (power moments), a, b
  constexpr int V_BK = (TRIG ? 2 : 1) * NL + 2, NV = V_BK + K + (TRIG ? 4 : 8);
  float own[NV];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    if constexpr (TRIG) {
      own[i] = TL.re[i];
      own[NL + i] = TL.im[i];
    } else {
      own[i] = L.l[i];
    }
  }
  own[V_BK - 2] = m0;
  own[V_BK - 1] = lam;
#pragma unroll
  for (int k = 1; k <= K; ++k) own[V_BK - 1 + k] = bk[k];
  if constexpr (!TRIG) {
    own[V_BK + K] = pb.tc;
    own[V_BK + K + 1] = pb.p;
    own[V_BK + K + 2] = pb.p15;
    own[V_BK + K + 3] = pb.amp;
  }
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) own[NV - 4 + ch] = ga[ch];
  own[NV - 1] = gb;
  rows.template put<NV>(lane, own);
  {
    // the window's pairs: gr their gradients, res their adjoint moments
    auto evaluate = [&](const Window& w, int& j, float* gr, float* res) __attribute__((always_inline)) {
      int p;
      const bool act = item_of(w, j, p);
      float pv[NV];
      rows.template get<NV>(p, own, pv);
      PixelBasis pp;
      LInv<NH> Lp;
      TrigLInv<TRIG ? NH : 1> TLp;
      if constexpr (TRIG) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          TLp.re[i] = pv[i];
          TLp.im[i] = pv[NL + i];
        }
      } else {
#pragma unroll
        for (int i = 0; i < NL; ++i) Lp.l[i] = pv[i];
        pp.tc = pv[V_BK + K];
        pp.p = pv[V_BK + K + 1];
        pp.p15 = pv[V_BK + K + 2];
        pp.amp = pv[V_BK + K + 3];
      }
      const float m0p = pv[V_BK - 2], lamp = pv[V_BK - 1];
      const float* bkp = pv + V_BK - 1;  // bkp[k], k = 1..K
      const float *gap = pv + NV - 4, gbp = pv[NV - 1];
      const float gpp = want_gp ? from_lane(gpen, p) : 0.f;
#pragma unroll
      for (int f = 0; f < G_COUNT; ++f) gr[f] = 0.f;
      if (act) {
        float dx, dy;
        offsets_of(j, p, dx, dy);
        RayG g = ray_params(st, j, dx, dy, lamp);
        QuadState<NH, NQ> s;
        TrigCanon<NH> tc[TRIG ? NQ : 1];
        int src[NQ];
        if constexpr (TRIG) {
          trig_quad_state<NH, NQ>(g, TLp, m0p, tn, a, s, tc, src);
        } else {
          quad_state<NH, NQ>(g, pp, Lp, m0p, tn, a, s);
        }
        float4 f5 = st.word(5, j);
        float gbar = gap[0] * f5.y + gap[1] * f5.z + gap[2] * f5.w + gbp;
        // consistency penalty (App. E): dP/dtau at the edges (bq, scaled by the
        // pixel's dL/dP) and its direct dependence on (mu, Sigma, omega)
        // through tau_ij = omega Sigma sqrt(pi/2) (erfc(b_j) - erfc(b_{j+1}))
        float bq[NQ];
#pragma unroll
        for (int e = 0; e < NQ; ++e) bq[e] = 0.f;
        float gmu = 0.f, gsig = 0.f, gom = 0.f;
        if (want_gp) {
          bool any_cl = false;
#pragma unroll
          for (int e = 0; e < NQ; ++e) any_cl = any_cl || s.cl[e];
          const float isg = fast_rcp(g.sig);
          const float bnear = (tn - g.mu) * kInvSqrt2 * isg;
          const float en = any_cl ? erfc_fast(bnear) : 0.f;
          const float gn = any_cl ? 1.1283791670955126f * __expf(-bnear * bnear) : 0.f;  // -d erfc / db
          const float cs = g.omega * g.sig * kSqrtHalfPi;
#pragma unroll
          for (int e = 0; e + 1 < NQ; ++e) {
            const float e0 = s.cl[e] ? en : a.ecq[e], e1 = s.cl[e + 1] ? en : a.ecq[e + 1];
            const float r = fmaxf(cs * (e0 - e1) - (s.tau[e + 1] - s.tau[e]), 0.f);
            const float tr = 2.f * r * gpp;
            bq[e] += tr;
            bq[e + 1] -= tr;
            const float ds0 = s.cl[e] ? gn * bnear * isg : 0.f, ds1 = s.cl[e + 1] ? gn * bnear * isg : 0.f;
            const float dm0 = s.cl[e] ? gn * kInvSqrt2 * isg : 0.f, dm1 = s.cl[e + 1] ? gn * kInvSqrt2 * isg : 0.f;
            gom += tr * g.sig * kSqrtHalfPi * (e0 - e1);
            gsig += tr * (g.omega * kSqrtHalfPi * (e0 - e1) + cs * (ds0 - ds1));
            gmu += tr * cs * (dm0 - dm1);
          }
        }
        float d[K + 1], gt[NQ];
#pragma unroll
        for (int k = 0; k <= K; ++k) d[k] = 0.f;
        // (radiance + penalty) gradient at fixed moments: through tau at the
        // edges (which move with mu and Sigma) and the Eq. 7 interval terms
        if constexpr (TRIG) {
          // dL/dtau gathered onto the edges whose queries supplied it
          float wsrc[NQ];
#pragma unroll
          for (int e = 0; e < NQ; ++e) wsrc[e] = 0.f;
#pragma unroll
          for (int e = 0; e < NQ; ++e) {
#pragma unroll
            for (int e2 = 0; e2 <= e; ++e2) wsrc[e2] += src[e] == e2 ? gbar * s.A[e] + bq[e] : 0.f;
          }
#pragma unroll
          for (int e = 0; e < NQ; ++e) {
            float gk[K + 1], dpsi;
            trig_adjoint<NH>(s.y[e], tc[e], a.beta, gk, dpsi);
            const float wgt = wsrc[e];
#pragma unroll
            for (int k = 1; k <= K; ++k) d[k] += wgt * gk[k];
            d[0] += wgt * s.F[e];
            const float dtau_dt = m0p * dpsi * kTrigSpan * warp_abs_d(s.t[e], tn);
            gt[e] = rounded(wgt * dtau_dt);
          }
        } else {
#pragma unroll
          for (int e = 0; e < NQ; ++e) {
            float lamk[2 * NH + 1], dl;
            hermite_adjoint<NH>(s.y[e], s.x[e], s.below[e], a.beta, lamk, dl);
            float wgt = gbar * s.A[e] + bq[e];
#pragma unroll
            for (int k = 1; k <= K; ++k) d[k] += wgt * lamk[k];
            d[0] += wgt * s.F[e];  // minus sum_k b_k d[k], taken once after the edges
            float dtau_dt = -m0p * s.w0[e] * dl * warp_dy(pp, s.t[e]);
            gt[e] = rounded(wgt * dtau_dt);
          }
        }
        edge_position_grads<NH, NQ>(s, a, gt, gmu, gsig);
#pragma unroll
        for (int k = 1; k <= K; ++k) d[0] -= bkp[k] * d[k];  // the tau = m_0 F(b) chain at b = m / m_0
        float dq0, dq1, dq2;
        quad_position_grads<NH, NQ>(g, s, a, dq0, dq1, dq2);
        gmu += gbar * dq0;
        gsig += gbar * dq1;
        gom += gbar * dq2;
        Results<K + 1> r;
#pragma unroll
        for (int k = 0; k <= K; ++k) r.v[k] = d[k];
        r.store(res, lane);
        chain_record(gmu, gsig, gom, g, lamp, dx, dy, st.word(2, j), st.word(3, j), st.word(4, j), gr);
        gr[G_CR] = s.q * gap[0];
        gr[G_CG] = s.q * gap[1];
        gr[G_CB] = s.q * gap[2];
      }
    };
    auto add_own = [&](uint64_t own, const float* res) __attribute__((always_inline)) {
      for_each_own(
          own,
          [&](int i) __attribute__((always_inline)) {
            Results<K + 1> r;
            r.load(res, i);
            return r;
          },
          [&](const Results<K + 1>& r) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k <= K; ++k) dm[k] += r.v[k];
          });
    };
    auto flush = [&](const Window& w) __attribute__((always_inline)) {
      int j;
      float gr[G_COUNT];
      evaluate(w, j, gr, res);
      __builtin_amdgcn_wave_barrier();
      add_own(w.own, res);
      reduce_to_slots<false>(w, gr, j, lane, cw, ba.partials, st, quad);
    };
    // each wave its window of the group, then the adjoint moments in window order
    // by every wave; a sum carried into wave 0's window is the group before's
    auto flush_group = [&](const Group& g) __attribute__((always_inline)) {
      const Window w = g.window(wave);
      int j = 0;
      float gr[G_COUNT], carried[G_COUNT];
      if (w.n > 0) {
        evaluate(w, j, gr, wres[4 * par + wave]);
        scan_window<false>(w, gr);
        leave_carry(w, gr, lane, carry[4 * par + wave]);
        if (wave == 0 && w.carried)
#pragma unroll
          for (int f = 0; f < G_COUNT; ++f) carried[f] = carry[4 * (par ^ 1) + 3][f];
      }
      __syncthreads();
      if (w.n > 0) {
        take_carry(w, gr, lane, wave == 0 ? carried : carry[4 * par + wave - 1]);
        write_slots<false>(w, gr, j, ba.partials, st, quad);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (g.n > 64 * k) add_own(g.own[k], wres[4 * par + k]);
      par ^= 1;
    };
    for (int b = rg.x; b < rg.y; b += kBlock) {
      int nb = min(kBlock, rg.y - b);
      stage(b, nb, true);
      if (wide) {
        if constexpr (WIDE)
          walk_groups<true>(ring[wave], a.masks, b, nb, quad, lane, active_mask, flush_group, [&](int j) {
            if (wave == 0) zero_slot(j);
          });
      } else {
        walk_entries<true>(q, a.masks, b, nb, quad, own4, lane, active_mask, flush, zero_slot);
      }
    }
  }

  }
  if (split) {
    float* xf = reinterpret_cast<float*>(&st);
    __syncthreads();
#pragma unroll
    for (int k = 0; k <= K; ++k) xf[(wave * (K + 1) + k) * 64 + lane] = dm[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k <= K; ++k) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) t += xf[(w * (K + 1) + k) * 64 + lane];
      dm[k] = t;
    }
  }

  if (!SUR && __ballot(active && mix_eps != 0.f) != 0) {
    // (b is formed again: few pixels come here, and it is not kept through the passes)
    if (active && mix_eps != 0.f) {
#pragma unroll
      for (int k = 1; k <= K; ++k) bk[k] = (float)(a.pix_mom[(size_t)k * a.n_pix + pix] / a.pix_mom[pix]);
    }
  }
  if (!SUR && active && mix_eps != 0.f) {
    // a degenerate pixel: the pairs took dL/db' at the mixture b' (dm[1..K]);
    // back to b through the mixture, and dm[0]'s share -sum_k b_k dL/db_k
    // follows the changed dL/db. With the identity factor F does not depend
    // on b, and the moments pass no gradient but m_0's.
    double bn[K + 1], D[K + 1];
    bn[0] = 1.0;
    D[0] = 0.0;
#pragma unroll
    for (int k = 1; k <= K; ++k) {
      bn[k] = (double)bk[k];
      D[k] = dm[k];
    }
    if (mix_eps > 0.f) {
      if constexpr (TRIG) {
        // mixed with the uniform measure on the circle: c' = (1 - eps) c + eps e_0
#pragma unroll
        for (int k = 1; k <= K; ++k) D[k] *= 1.0 - (double)mix_eps;
      } else {
        mixture_adjoint<K + 1>(bn, (double)mix_eps, D);
      }
    } else {
#pragma unroll
      for (int k = 1; k <= K; ++k) D[k] = 0.0;
    }
    double corr = 0.0;
#pragma unroll
    for (int k = 1; k <= K; ++k) corr += (double)bk[k] * ((double)dm[k] - D[k]);
    dm[0] += (float)corr;
#pragma unroll
    for (int k = 1; k <= K; ++k) dm[k] = (float)D[k];
  }

  // ---- pass 3: the moment part of the Gradient stage ------------------------
  constexpr int NV3 = K + 2 + (TRIG ? 0 : 4);  // dm, lambda, basis
  static_assert(NV3 <= S, "pass 3 takes all values from LDS");
  {
    float own[NV3];
#pragma unroll
    for (int k = 0; k <= K; ++k) own[k] = dm[k];
    own[K + 1] = lam;
    if constexpr (!TRIG) {
      own[K + 2] = pb.tc;
      own[K + 3] = pb.p;
      own[K + 4] = pb.p15;
      own[K + 5] = pb.amp;
    }
    if constexpr (WIDE) __syncthreads();  // the rows are the four waves'
    rows.template put<NV3>(lane, own);
  }
  {
    auto evaluate = [&](const Window& w, int& j, float* gr, SlotVals& prev) __attribute__((always_inline)) {
      int p;
      const bool act = item_of(w, j, p);
      prev = load_slot(w, j, ba.partials, st, quad);
      float pv[NV3];
      rows.template get<NV3>(p, nullptr, pv);
      const float* dmp = pv;
      const float lamp = pv[K + 1];
      PixelBasis pp;
      if constexpr (!TRIG) {
        pp.tc = pv[K + 2];
        pp.p = pv[K + 3];
        pp.p15 = pv[K + 4];
        pp.amp = pv[K + 5];
      }
#pragma unroll
      for (int f = 0; f < G_COUNT; ++f) gr[f] = 0.f;
      if (act) {
        float dx, dy;
        offsets_of(j, p, dx, dy);
        RayG g = ray_params(st, j, dx, dy, lamp);
        float gm[3];
        if constexpr (TRIG)
          trig_moment_grads<NH>(g, tn, dmp, gm);
        else
          moment_grads<K>(g, pp, tn, dmp, gm);
        chain_record(gm[0], gm[1], gm[2], g, lamp, dx, dy, st.word(2, j), st.word(3, j), st.word(4, j), gr);
      }
    };
    auto flush = [&](const Window& w) __attribute__((always_inline)) {
      int j;
      float gr[G_COUNT];
      SlotVals prev;
      evaluate(w, j, gr, prev);
      reduce_to_slots<true>(w, gr, j, lane, cw, ba.partials, st, quad, &prev);
    };
    auto flush_group = [&](const Group& g) __attribute__((always_inline)) {
      const Window w = g.window(wave);
      int j = 0;
      float gr[G_COUNT], carried[G_COUNT];
      SlotVals prev;
      if (w.n > 0) {
        evaluate(w, j, gr, prev);
        scan_window<true>(w, gr);
        leave_carry(w, gr, lane, carry[4 * par + wave]);
        if (wave == 0 && w.carried)
#pragma unroll
          for (int f = 0; f < G_COUNT; ++f) carried[f] = carry[4 * (par ^ 1) + 3][f];
      }
      __syncthreads();
      if (w.n > 0) {
        take_carry(w, gr, lane, wave == 0 ? carried : carry[4 * par + wave - 1]);
        write_slots<true>(w, gr, j, ba.partials, st, quad, &prev);
      }
      par ^= 1;
    };
    for (int b = rg.x; b < rg.y; b += kBlock) {
      int nb = min(kBlock, rg.y - b);
      stage(b, nb, false);
      if (wide) {
        if constexpr (WIDE)
          walk_groups<false>(ring[wave], a.masks, b, nb, quad, lane, active_mask, flush_group, [](int) {});
      } else {
        walk_entries<false>(q, a.masks, b, nb, quad, own4, lane, active_mask, flush, [](int) {});
      }
    }
  }
}

hipError_t launch_render_backward(const RenderArgs& r, const float* saved, const float* grad_image,
                                  const float* grad_penalty, const int* sorted_k, float* partials,
                                  uint8_t* used, const CamSet& cams, int n_moments, int n_intervals,
                                  hipStream_t s, int mode) {
  BwdArgs ba{r, saved, grad_image, grad_penalty, sorted_k, partials, used};
  int n_keys = r.tiles_x * r.tiles_y * r.n_cams;
  dim3 grid(render_blocks(n_keys)), block(kBlock);
#define MB_LAUNCH_WIDE(KK, NN, SS)                                                                           \
  if (wide && n_moments == KK && n_intervals == NN && mode == SS) {                                          \
    hipLaunchKernelGGL((k_render_bwd<KK, NN + 1, SS, true>), dim3(4 * n_keys), block, 0, s, ba, cams);       \
    return hipGetLastError();                                                                                \
  }
  // (not the trigonometric K = 6, whose sums follow the compiler's choice of fused
  // operations in the last bit)
  const bool wide = n_keys <= kWideTiles;
  MB_LAUNCH_WIDE(4, 3, 0)
  MB_LAUNCH_WIDE(6, 3, 0)
  MB_LAUNCH_WIDE(4, 5, 0)
  MB_LAUNCH_WIDE(6, 5, 0)
  MB_LAUNCH_WIDE(8, 3, 0)
  MB_LAUNCH_WIDE(8, 5, 0)
  MB_LAUNCH_WIDE(4, 3, 2)
  MB_LAUNCH_WIDE(4, 5, 2)
#undef MB_LAUNCH_WIDE
#define MB_LAUNCH(KK, NN, SS)                                                          \
  if (n_moments == KK && n_intervals == NN && mode == SS) {                            \
    hipLaunchKernelGGL((k_render_bwd<KK, NN + 1, SS>), grid, block, 0, s, ba, cams); \
    return hipGetLastError();                                                          \
  }
  MB_LAUNCH(4, 3, 0)
  MB_LAUNCH(6, 3, 0)
  MB_LAUNCH(4, 5, 0)
  MB_LAUNCH(6, 5, 0)
  MB_LAUNCH(8, 3, 0)
  MB_LAUNCH(8, 5, 0)
  MB_LAUNCH(6, 3, 1)
  MB_LAUNCH(6, 5, 1)
  MB_LAUNCH(4, 3, 2)
  MB_LAUNCH(4, 5, 2)
  MB_LAUNCH(6, 3, 2)
  MB_LAUNCH(6, 5, 2)
#undef MB_LAUNCH
  return hipErrorInvalidValue;
}

}  // namespace mb
