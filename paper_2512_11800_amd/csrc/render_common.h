// Per-pair building blocks shared by the forward and backward render
// kernels: LDS staging of render records, the coverage test, the ray-space
// Gaussian, the warped moments and the per-Gaussian quadrature.
#pragma once
#include "kernels.h"
#include "recon.h"

namespace mb {

struct Stage {
  float4 f[kRecF4][kBlock];
  __device__ __forceinline__ const float4& word(int k, int j) const { return f[k][j]; }
};

struct RayG {
  float mu, sig, omega;
  float id, xid, ek;  // 1 / D, X / D and exp(-X / 2D) at the pixel offset (for the adjoint)
  float le;           // mu D
};

// ---------------------------------------------------------------------------
// Per-wave compaction of covering pairs. A wave owns an 8x8 pixel block; while
// it walks the stored coverage masks, (entry, pixel) pairs are appended to a queue,
// all of them entry by entry (walk_entries) or those of thin rounds (walk_pairs), and
// evaluated 64 at a time, one pair per lane, so the arithmetic runs on full waves
// whatever the fraction of the block a Gaussian covers. A pair's results go back to
// the pixel's own lane (the owner), which adds them in queue order: per pixel the
// summation order is the list order, as without compaction.
// ---------------------------------------------------------------------------
struct WaveQueue {
  uint16_t item[128];  // (entry in the staged batch) << 6 | pixel lane
};

struct QueueCursor {
  int cnt;                  // queued pairs (wave-uniform)
  uint64_t own_lo, own_hi;  // this lane's queue positions [0, 64) and [64, 128)
};

__device__ __forceinline__ void queue_reset(QueueCursor& qc) {
  qc.cnt = 0;
  qc.own_lo = 0;
  qc.own_hi = 0;
}

// After evaluating positions [0, 64): move the rest to the front.
__device__ __forceinline__ void queue_pop64(WaveQueue& q, QueueCursor& qc, int lane) {
  int rest = qc.cnt - 64;
  uint16_t it = lane < rest ? q.item[64 + lane] : (uint16_t)0;
  __builtin_amdgcn_wave_barrier();
  if (lane < rest) q.item[lane] = it;
  __builtin_amdgcn_wave_barrier();
  qc.own_lo = qc.own_hi;
  qc.own_hi = 0;
  qc.cnt = rest;
}

// value of pixel lane p (all lanes must take part)
__device__ __forceinline__ float from_lane(float v, int p) { return __shfl(v, p, 64); }

// Work of a render block (see launch_tile_order): tile key (camera * tiles +
// tile; n_keys or more for an empty block) and, for a block of a split tile, the
// quadrant its four waves share (quad = -1: the whole tile, one quadrant per
// wave).
struct BlockWork {
  int key, quad;
};
__device__ __forceinline__ BlockWork block_work(const RenderArgs& a) {
  const int code = a.order[blockIdx.x];
  BlockWork w;
  if (code >= 0) {
    w.key = code;
    w.quad = -1;
  } else {
    const int v = -code - 1;
    w.key = v >> 2;
    w.quad = v & 3;
  }
  return w;
}

// The blocks of the kernels' wide form for frames of few tiles: the split tiles' as in the block list, then four for each
// other tile in its order.
struct WideWork {
  int key, quad;
  bool split;
};
__device__ __forceinline__ WideWork wide_work(const RenderArgs& a, int n_keys) {
  const int last = a.order[render_blocks(n_keys) - 1];
  const int ns = last < 0 ? n_keys : last - n_keys;  // split tiles
  const int b = (int)blockIdx.x, i = (b >> 2) - ns;
  WideWork w;
  w.quad = b & 3;
  w.split = i < 0;
  w.key = w.split ? (-a.order[b] - 1) >> 2 : a.order[4 * ns + i];
  return w;
}

__device__ __forceinline__ void load_batch(Stage& st, const float4* rec, const int* sorted_rec, int b, int nb) {
  int tid = threadIdx.x;
  if (tid < nb) {
    const float4* src = rec + (size_t)sorted_rec[b + tid] * kRecStride;
#pragma unroll
    for (int k = 0; k < kRecF4; ++k) st.f[k][tid] = src[k];
  }
}

// load_batch for the passes that walk the stored coverage masks: an entry
// whose masks are empty for every quadrant the block renders is never
// evaluated, so its record is not fetched (its staging slot keeps stale
// data that nothing reads). quad >= 0: a split block's one quadrant; -1: the
// whole tile (any of the four masks).
__device__ __forceinline__ void load_batch_covered(Stage& st, const float4* rec, const int* sorted_rec,
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
#pragma unroll
      for (int k = 0; k < kRecF4; ++k) st.f[k][tid] = src[k];
    }
  }
}

// Coverage of the pixel centres of a tile by staged entry j, in the
// rectangle's axis coordinates c1 = (p - C) . e1, c2 = (p - C) . e2 (C, e1,
// e2 = e1 rotated by +90 degrees, halves h1, h2 from the record; covered iff
// |c1| <= h1 and |c2| <= h2). cover_setup evaluates (c1, c2) once per entry at
// the tile's first pixel centre (x_t + 1/2, y_t + 1/2); the per-pixel test
// adds the pixel's offset (i, j) inside the tile, c1 + i e1x + j e1y and
// c2 - i e1y + j e1x, two fused multiply-adds each. The float test decides
// wherever its margin to an edge exceeds `band`, a bound on its rounding
// error: the record's centre offset, axis and halves are the double values
// rounded to float (relative 2^-24), and the set-up and per-pixel operations
// round relative 2^-24 each; summed, the error stays below
// 2^-24 (9 (|a_x| + |a_y|) + 2 (|o_x| + |o_y|) + 2 (h1 + h2) + 100) (a: the
// tile origin's offset from the rectangle's centre, o: the centre's offset
// from the projected mean), and the band 1e-6 (16 + |a_x| + |a_y| + |o_x| +
// |o_y| + h1 + h2) is about twice that. An entry with a pixel inside its band
// is tested again by the whole wave, those pixels in double against rectd.
// Only the first pass tests coverage: every later pass, forward and backward,
// reads the masks it stores.
//
// The set-up lives in LDS the kernel already holds: (c1, c2) at the tile
// origin replace the staged record's centre offset (st.f[0][j].zw, which
// the first pass reads nowhere else). Returns the band.
__device__ __forceinline__ float cover_setup(Stage& st, int j, int xt, int yt) {
  const float4 f0 = st.f[0][j], f1 = st.f[1][j];
  const float ax = ((float)xt + 0.5f - f0.x) - f0.z;
  const float ay = ((float)yt + 0.5f - f0.y) - f0.w;
  const float a1 = ax * f1.x + ay * f1.y;
  const float a2 = ay * f1.x - ax * f1.y;
  st.f[0][j] = make_float4(f0.x, f0.y, a1, a2);
  return 1e-6f * (16.f + fabsf(ax) + fabsf(ay) + fabsf(f0.z) + fabsf(f0.w) + f1.z + f1.w);
}

// The 64 pixels of the tile's 8x8 block `quad` that entry j covers (bit
// 8 row + column), one entry per lane (after cover_setup), by the float test;
// `near` receives the smallest margin to an edge among them. One lane per
// entry shares an entry's set-up over its 64 tests and leaves the mask where
// it is stored from: about 24 issue cycles an entry, where the wave testing
// one entry with a lane per pixel took about 90 (uniform reads, ballot and
// a store for each).
__device__ __forceinline__ uint64_t cover_entry(const Stage& st, int j, int quad, float& near) {
  const float4 f0 = st.f[0][j], f1 = st.f[1][j];
  float p1[8], p2[8];  // the columns' part of (c1, c2)
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float fi = (float)(8 * (quad & 1) + i);
    p1[i] = fmaf(fi, f1.x, f0.z);
    p2[i] = fmaf(fi, -f1.y, f0.w);
  }
  near = 1e30f;
  uint32_t out[2];
#pragma unroll
  for (int h = 1; h >= 0; --h) {
    uint32_t bits = 0;  // the tests' sign bits (1: outside), the last pixel first
    // a row at a time: unrolled further, the compiler keeps all 64 tests' values live
#pragma unroll 1
    for (int r = 3; r >= 0; --r) {
      float fj = (float)(8 * (quad >> 1) + 4 * h + r);
      asm("" : "+v"(fj));  // in a vector register: a scalar operand halves the rate of fp32 multiply-adds
#pragma unroll
      for (int i = 7; i >= 0; --i) {
        const float c1 = fmaf(fj, f1.y, p1[i]), c2 = fmaf(fj, f1.x, p2[i]);
        const float m = fminf(f1.z - fabsf(c1), f1.w - fabsf(c2));
        near = fminf(near, fabsf(m));
        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(m), 31);
      }
    }
    out[h] = ~bits;
  }
  return ((uint64_t)out[1] << 32) | out[0];
}

// The same test of one entry j by the whole wave, one pixel per lane (offset
// (fi, fj) from the tile's first pixel, centre (u, v)), with the pixels inside
// the band decided in double.
__device__ __forceinline__ bool covers(const Stage& st, float band, const double2* rectd, const int* sorted_rec,
                                       int b, int j, float fi, float fj, float u, float v) {
  const float4 f0 = st.f[0][j], f1 = st.f[1][j];
  const float c1 = fmaf(fj, f1.y, fmaf(fi, f1.x, f0.z));
  const float c2 = fmaf(fj, f1.x, fmaf(fi, -f1.y, f0.w));
  const float m = fminf(f1.z - fabsf(c1), f1.w - fabsf(c2));
  bool cov = m >= 0.f;
  if (fabsf(m) < band) {
    const int rid = __builtin_amdgcn_readfirstlane(sorted_rec[b + j]);
    const double2 cd = rectd[(size_t)rid * 3], ed = rectd[(size_t)rid * 3 + 1], hd = rectd[(size_t)rid * 3 + 2];
    const double axd = (double)u - cd.x, ayd = (double)v - cd.y;
    const double c1d = axd * ed.x + ayd * ed.y;
    const double c2d = -axd * ed.y + ayd * ed.x;
    cov = fabs(c1d) <= hd.x && fabs(c2d) <= hd.y;
  }
  return cov;
}

// 64 x 64 bit transpose over the wave: from the coverage masks of 64 entries
// (lane = entry, bit = pixel) the words of 64 pixels (lane = pixel, bit =
// entry), and back. Six exchanges with lane ^ s, s = 32, 16, .., 1: a lane
// keeps the bits whose index agrees with its own in bit s and takes the others
// from its partner, shifted by s. About 200 issue cycles.
__device__ __forceinline__ uint64_t transpose_masks(uint64_t m, int lane) {
  uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
  {
    // s = 32: the upper lanes' low words change places with the lower lanes' high words
    const uint32_t give = lane & 32 ? lo : hi;
    const uint32_t got = (uint32_t)__shfl_xor((int)give, 32, 64);
    lo = lane & 32 ? got : lo;
    hi = lane & 32 ? hi : got;
  }
  auto step = [&](uint32_t plo, uint32_t phi, int s, uint32_t mask) __attribute__((always_inline)) {
    const uint32_t keep = lane & s ? ~mask : mask;
    const uint32_t rot = lane & s ? (uint32_t)s : (uint32_t)(32 - s);
    lo = (lo & keep) | (__builtin_amdgcn_alignbit(plo, plo, rot) & ~keep);
    hi = (hi & keep) | (__builtin_amdgcn_alignbit(phi, phi, rot) & ~keep);
  };
  step((uint32_t)__builtin_amdgcn_ds_swizzle((int)lo, 0x401F), (uint32_t)__builtin_amdgcn_ds_swizzle((int)hi, 0x401F),
       16, 0x0000FFFFu);
  step((uint32_t)__builtin_amdgcn_mov_dpp((int)lo, 0x128, 0xF, 0xF, true),
       (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, 0x128, 0xF, 0xF, true), 8, 0x00FF00FFu);  // row_ror:8
  step((uint32_t)__builtin_amdgcn_ds_swizzle((int)lo, 0x101F), (uint32_t)__builtin_amdgcn_ds_swizzle((int)hi, 0x101F),
       4, 0x0F0F0F0Fu);
  step((uint32_t)__builtin_amdgcn_mov_dpp((int)lo, 0x4E, 0xF, 0xF, true),
       (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, 0x4E, 0xF, 0xF, true), 2, 0x33333333u);  // quad_perm 2,3,0,1
  step((uint32_t)__builtin_amdgcn_mov_dpp((int)lo, 0xB1, 0xF, 0xF, true),
       (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, 0xB1, 0xF, 0xF, true), 1, 0x55555555u);  // quad_perm 1,0,3,2
  return ((uint64_t)hi << 32) | lo;
}

// Walks of a staged batch [b, b + nb) by pixel words (lane = pixel, bit =
// entry), 64 entries (a chunk) at a time. A wave takes all the batch's chunks
// of consecutive entries; in a split block (see BlockWork) it takes every
// fourth entry, one chunk a batch (`own4` >= 0: its index). A round takes one
// entry from every lane that has entries left, each its own: the lane holds its
// pixel's values and sums in its registers, so nothing is queued, broadcast or
// sent back, and every pixel's sums run in list order.
__device__ __forceinline__ int n_chunks(int nb, int own4) { return own4 < 0 ? (nb + 63) >> 6 : 1; }
// Entry of the staged batch that bit (or lane) e of chunk c stands for.
__device__ __forceinline__ int chunk_entry(int c, int e, int own4) { return own4 < 0 ? 64 * c + e : 4 * e + own4; }
// Coverage masks of chunk c, one entry per lane.
__device__ __forceinline__ uint64_t load_masks(const uint64_t* masks, int b, int nb, int quad, int own4, int c,
                                               int lane) {
  const int j = chunk_entry(c, lane, own4);
  return j < nb ? masks[(size_t)(b + j) * 4 + quad] : 0ull;
}
// body(j) for the entries of this lane's word m of chunk c (no cross-lane
// operations in it): 64 pairs take 1.38 rounds in the case step_1080p of perf/cases.py,
// for the pixels of a block have unequal counts.
template <class Body>
__device__ __forceinline__ void word_rounds(uint64_t m, int c, int own4, Body&& body) {
  while (m != 0) {
    const int e = __builtin_ctzll(m);
    m &= m - 1;
    body(chunk_entry(c, e, own4));
  }
}
// The rounds over the stored masks, for the lanes with `live`.
template <class Body>
__device__ __forceinline__ void for_each_own_entry(const uint64_t* masks, int b, int nb, int quad, int own4, int lane,
                                                   bool live, Body&& body) {
  const int nc = n_chunks(nb, own4);
  uint64_t next = load_masks(masks, b, nb, quad, own4, 0, lane);
  for (int c = 0; c < nc; ++c) {
    const uint64_t w = transpose_masks(next, lane);
    if (c + 1 < nc) next = load_masks(masks, b, nb, quad, own4, c + 1, lane);
    word_rounds(live ? w : 0ull, c, own4, body);
  }
}

// The same rounds for an evaluation that costs far more than queueing a pair:
// a round with kDirectLanes lanes or more is evaluated as it stands, and the
// pairs of the thinner rounds are queued and evaluated 64 at a time, one per
// lane, their results sent back to the pixel's own lane. The queue is emptied at
// the end of each chunk, so a pixel's results still arrive in list order. In the
// case step_1080p 86% of the pairs are evaluated directly, 97% of
// their lanes at work; all rounds direct would leave 73% at work, all pairs
// queued cost a push, thirteen broadcasts and an owner sum each.
// eval(direct, on, j, p, own): one evaluation for the lanes with `on`, of entry
// j at pixel lane p; direct (wave-uniform): p is the lane itself; otherwise
// bits of `own` are the lanes whose results belong to this lane's pixel. All
// lanes call it.
constexpr int kDirectLanes = 48;
template <class Eval>
__device__ __forceinline__ void walk_pairs(WaveQueue& q, const uint64_t* masks, int b, int nb, int quad, int own4,
                                           int lane, bool live, Eval&& eval) {
  const int nc = n_chunks(nb, own4);
  int c = -1;
  uint64_t next = load_masks(masks, b, nb, quad, own4, 0, lane);
  uint64_t m = 0;
  QueueCursor qc;
  queue_reset(qc);
  for (;;) {
    const uint64_t act = __ballot(m != 0);
    const int n = __popcll(act);
    if (n == 0 && qc.cnt == 0 && c + 1 < nc) {
      const uint64_t w = transpose_masks(next, lane);
      m = live ? w : 0ull;
      ++c;
      if (c + 1 < nc) next = load_masks(masks, b, nb, quad, own4, c + 1, lane);
      continue;
    }
    const bool direct = n >= kDirectLanes;
    int j = 0, p = lane;
    bool on = m != 0;
    if (on) {
      j = chunk_entry(c, (int)__builtin_ctzll(m), own4);
      m &= m - 1;
    }
    if (!direct) {
      if (on) {
        const int pos = qc.cnt + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(act >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)act, 0u));
        q.item[pos] = (uint16_t)((j << 6) | lane);
        // bit pos of (own_lo, own_hi), by masks: chains of 64-bit selects on
        // the carry register issue five times slower than plain logic here
        const uint64_t bit = 1ull << (pos & 63);
        const uint64_t hi = 0ull - (uint64_t)(pos >> 6);
        qc.own_lo |= bit & ~hi;
        qc.own_hi |= bit & hi;
      }
      qc.cnt += n;
      if (qc.cnt < 64 && (n != 0 || qc.cnt == 0)) {
        if (n == 0) break;
        continue;
      }
      __builtin_amdgcn_wave_barrier();
      on = lane < qc.cnt;
      const int it = on ? (int)q.item[lane] : lane;
      j = it >> 6;
      p = it & 63;
    }
    eval(direct, on, j, p, qc.own_lo);
    if (!direct) {
      if (qc.cnt > 64) {
        queue_pop64(q, qc, lane);
      } else {
        queue_reset(qc);
      }
    }
  }
}

// A queue of pairs, entry by entry (in the backward pass pairs of one entry lie next
// to each other so that a segmented scan over the lanes sums an entry's gradients; in
// the forward pass of trigonometric K = 6 for their alike iterations): positions [0, 64) are the window evaluated next. Everything but
// the lanes' own positions is wave-uniform and kept in scalar registers: an entry
// is queued under its mask as the execution mask, and the window's segments come
// from `heads` by scalar logic. Masks fetched with a shuffle, a count in vector
// registers and a lane's positions by 64-bit selects cost a push about 150 issue
// cycles, against 50 (2.9 pushes per 64 pairs and pass in the case step_1080p).
struct Window {
  int n;           // pairs in the window
  int base;        // its first item in the ring of 128
  uint64_t heads;  // positions that begin an entry's pairs
  uint64_t own;    // this lane's positions: the pairs of its pixel
  bool carried;    // the first segment continues the entry of the window before
  bool continues;  // the last segment's entry continues in the next window
};

// Rank tracking beside a queue: q[item] receives the pair's index among its
// pixel's covering pairs, counted by the pixel lane's ctr.
struct QueueRanks {
  uint32_t* q;  // [128] in LDS, parallel to WaveQueue::item
  uint32_t ctr;
};

// Queue the pairs of the staged batch [b, b + nb) from the stored coverage masks of
// this wave (restricted to the lanes of `keep`), skipping empty entries 64 at a
// time, and call flush(window) for every 64 pairs and for the rest. on_empty(j) is
// called by the lane that loaded entry j's mask when the stored mask has pixels but
// none of them is kept. In a split block (see BlockWork) a wave takes only the
// entries j with j % 4 == its wave index (`own4` >= 0); otherwise every entry.
// OWN: the lanes' own positions are wanted.
template <bool OWN, class Flush, class Empty>
__device__ __forceinline__ void walk_entries(WaveQueue& q, const uint64_t* masks, int b, int nb, int quad, int own4,
                                             int lane, uint64_t keep, Flush&& flush, Empty&& on_empty,
                                             QueueRanks* rank = nullptr) {
  Window w = {0, 0, 0ull, 0ull, false, false};
  for (int j0 = 0; j0 < nb; j0 += 64) {
    const bool in = j0 + lane < nb && (own4 < 0 || ((j0 + lane) & 3) == own4);
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
      const int n = w.n + __builtin_popcountll(m);
      const bool cov = __builtin_amdgcn_inverse_ballot_w64(m);
      const uint16_t item = (uint16_t)(((j0 + l) << 6) | lane);
      w.heads |= 1ull << w.n;
      if (n < 64) {
        if (cov) {
          const int pos = (int)__builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, (uint32_t)w.n));
          q.item[w.base + pos] = item;
          if (rank) rank->q[w.base + pos] = rank->ctr++;
          if constexpr (OWN) w.own |= 1ull << pos;
        }
        w.n = n;
        continue;
      }
      uint64_t own_next = 0;  // at most one position past the window: an entry has one pair per pixel
      if (cov) {
        const int pos = (int)__builtin_amdgcn_mbcnt_hi(mhi, __builtin_amdgcn_mbcnt_lo(mlo, (uint32_t)w.n));
        const int at = (w.base + pos) & 127;
        q.item[at] = item;
        if (rank) rank->q[at] = rank->ctr++;
        if constexpr (OWN) {
          const uint64_t bit = 1ull << (pos & 63);
          if (pos < 64)
            w.own |= bit;
          else
            own_next = bit;
        }
      }
      w.n = 64;
      w.continues = n > 64;
      flush(w);
      w.carried = n > 64;
      w.n = n - 64;
      w.base ^= 64;
      w.heads = n > 64 ? 1ull : 0ull;
      w.own = own_next;
    }
  }
  w.continues = false;
  if (w.n > 0) flush(w);
}

// Eqs. 4-6 for the pixel ray in the projected-mean frame (see common.h)
template <class St>
__device__ __forceinline__ RayG ray_params(const St& st, int j, float dx, float dy, float lam) {
  float4 f2 = st.word(2, j), f3 = st.word(3, j), f4 = st.word(4, j);
  float w = st.word(5, j).x;
  float d = f2.x + 2.f * (f2.y * dx + f2.z * dy) + f2.w * dx * dx + 2.f * f3.x * dx * dy + f3.y * dy * dy;
  float e = f3.z + f3.w * dx + f4.x * dy;
  float x = f4.y * dx * dx + 2.f * f4.z * dx * dy + f4.w * dy * dy;
  float id = fast_rcp(d);
  RayG g;
  g.id = id;
  g.xid = x * id;
  g.ek = exp_neg_half(g.xid);
  g.le = lam * e;
  g.mu = g.le * id;
  g.sig = lam * fast_rsq(d);
  g.omega = w * g.ek;
  return g;
}

// warp_y with its fused operations fixed. Small pivots of the pixel's Hankel
// matrix magnify a moment's last bits, so the moments round the same way
// whatever code surrounds them.
__device__ __forceinline__ float warp_y_moment(const PixelBasis& b, float t, float dt) {
  const float q = fmaf(0.8f, t, 1.f);
  const float sq = fast_sqrt(q);
  const float num = fmaf(b.p, b.p, (q + b.p) * q);
  const float den = fmaf(q, sq, b.p15) * (b.p15 * (q * sq));
  return b.amp * dt * num * fast_rcp(den);
}

// warped moments of one ray Gaussian, Eqs. 10-12 (t_f -> inf), in the pixel's
// moment variable; the boundary term enters with '+' (App. C)
template <int K>
__device__ __forceinline__ void particle_moments(const RayG& g, const PixelBasis& pb, float tn, float* m) {
  float mus = fmaxf(g.mu, tn);
  float ys = warp_y_moment(pb, mus, mus - pb.tc);
  float yp = warp_dy(pb, mus);
  float gg = ys + yp * (g.mu - mus);
  float is = fast_rcp(g.sig);
  float bn = (tn - g.mu) * kInvSqrt2 * is;
  float e = __expf(-bn * bn);
  float s2 = g.sig * g.sig;
  m[0] = g.omega * g.sig * kSqrtHalfPi * erfc_fast(bn);
  float bnd = yp * g.omega * s2 * e;
  m[1] = gg * m[0] + bnd;
  float un = gg + yp * (tn - g.mu);
  float unp = un;
  float v2 = yp * yp * s2;
#pragma unroll
  for (int k = 2; k <= K; ++k) {
    m[k] = gg * m[k - 1] + (float)(k - 1) * v2 * m[k - 2] + bnd * unp;
    unp *= un;
  }
}

// The same moments with the recurrence in double (from the float ray
// Gaussian): each pair's moment vector is then, to double rounding, the exact
// moment vector of a Gaussian, so the pixel's Hankel matrix keeps its small
// pivots. Independent float rounding of the nine moments of K = 8 moves a
// pivot of 1e-5 (relative) by several percent, enough to shift the bounds.
template <int K>
__device__ __forceinline__ void particle_moments_d(const RayG& g, const PixelBasis& pb, float tn, double* m) {
  float mus = fmaxf(g.mu, tn);
  float ys = warp_y_moment(pb, mus, mus - pb.tc);
  float yp = warp_dy(pb, mus);
  const double gg = (double)ys + (double)yp * (double)(g.mu - mus);
  float is = fast_rcp(g.sig);
  float bn = (tn - g.mu) * kInvSqrt2 * is;
  float e = __expf(-bn * bn);
  const double s2 = (double)g.sig * (double)g.sig;
  m[0] = (double)(g.omega * g.sig * kSqrtHalfPi * erfc_fast(bn));
  const double bnd = (double)yp * (double)g.omega * s2 * (double)e;
  m[1] = gg * m[0] + bnd;
  const double un = gg + (double)yp * (double)(tn - g.mu);
  double unp = un;
  const double v2 = (double)yp * (double)yp * s2;
#pragma unroll
  for (int k = 2; k <= K; ++k) {
    m[k] = gg * m[k - 1] + (double)(k - 1) * v2 * m[k - 2] + bnd * unp;
    unp *= un;
  }
}

// phi(x) = (1 - e^-x) / x from d = e^-x: the Taylor series up to x^4 for
// |x| < 1/16 (truncation below 2e-9 relative), the direct form beyond (where
// 1 - d > 0.06, so its rounding stays below 1e-6 relative)
constexpr float kPhiSeries = 0.0625f;
__device__ __forceinline__ float phi_fn(float x, float d) {
  float s = 1.f / 120.f;
  s = fmaf(s, -x, 1.f / 24.f);
  s = fmaf(s, -x, 1.f / 6.f);
  s = fmaf(s, -x, 0.5f);
  s = fmaf(s, -x, 1.f);
  return fabsf(x) < kPhiSeries ? s : (1.f - d) * fast_rcp(x);
}

// x as it is: a product rounded here is not fused into a later sum
__device__ __forceinline__ float rounded(float x) {
  asm("" : "+v"(x));
  return x;
}

// Interval edges of one Gaussian's quadrature (App. B sample spacing): edge
// offsets, the clamp to the near bound, the moment variable y at each edge,
// the interval lengths and the particle density sigma_i at each edge.
template <int NQ>
struct QEdges {
  float off[NQ], y[NQ], sj[NQ], tau[NQ], delta[NQ - 1];
  bool cl[NQ];
};

template <int NQ>
__device__ __forceinline__ void quad_edges(const RayG& g, const PixelBasis& pb, float tn, const RenderArgs& a,
                                           QEdges<NQ>& e) {
  float dtc = g.mu - pb.tc;
  // every edge left of the near bound is moved onto it: one density there
  const float rn = (tn - g.mu) * fast_rcp(g.sig);
  const float en = exp_neg_half(rn * rn);
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    e.off[j] = a.kappa * g.sig * a.xq[j];
    float t = g.mu + e.off[j];
    e.cl[j] = t < tn;
    float dt = e.cl[j] ? (tn - pb.tc) : (dtc + e.off[j]);
    t = e.cl[j] ? tn : t;
    e.y[j] = warp_y(pb, t, dt);
    e.sj[j] = g.omega * (e.cl[j] ? en : a.eq[j]);
  }
}

// The same with the clamped edges' values formed only in waves that have one (the
// first edge is the nearest, so it tells; most Gaussians lie beyond the near
// bound).
template <int NQ>
__device__ __forceinline__ void quad_edges_far(const RayG& g, const PixelBasis& pb, float tn, const RenderArgs& a,
                                           QEdges<NQ>& e) {
  // the fused operations are fixed (rounded): the backward pass forms the same
  // edges, and its moment adjoint magnifies their last bits
  const float dtc = rounded(g.mu) - pb.tc;
  const float ks = a.kappa * g.sig;
  float t[NQ], dt[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    e.off[j] = rounded(ks * a.xq[j]);
    t[j] = fmaf(ks, a.xq[j], g.mu);
    dt[j] = dtc + e.off[j];
    e.sj[j] = g.omega * a.eq[j];
    e.cl[j] = t[j] < tn;
  }
#pragma unroll
  for (int j = 0; j + 1 < NQ; ++j) e.delta[j] = e.off[j + 1] - e.off[j];
  if (__ballot(e.cl[0]) != 0) {
    // every edge left of the near bound is moved onto it: one density there
    const float rn = (tn - g.mu) * fast_rcp(g.sig);
    const float en = g.omega * exp_neg_half(rn * rn);
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      dt[j] = e.cl[j] ? (tn - pb.tc) : dt[j];
      t[j] = e.cl[j] ? tn : t[j];
      e.sj[j] = e.cl[j] ? en : e.sj[j];
    }
#pragma unroll
    for (int j = 0; j + 1 < NQ; ++j)
      e.delta[j] = e.cl[j + 1] ? 0.f : (e.cl[j] ? t[j + 1] - tn : e.delta[j]);
  }
#pragma unroll
  for (int j = 0; j < NQ; ++j) e.y[j] = warp_y(pb, t[j], dt[j]);
}

// Eq. 7 sum over the intervals, given the optical depth at every edge
template <int NQ>
__device__ __forceinline__ float quad_sum(const RayG& g, float tn, const QEdges<NQ>& e) {
  float q = 0.f;
  float T = __expf(-e.tau[0]);  // transmittance at edge j, carried along the edges
#pragma unroll
  for (int j = 0; j + 1 < NQ; ++j) {
    float delta = e.cl[j + 1] ? 0.f : (e.cl[j] ? (g.mu + e.off[j + 1] - tn) : (e.off[j + 1] - e.off[j]));
    const float x = e.tau[j + 1] - e.tau[j];
    const float d = __expf(-x);
    q += T * delta * phi_fn(x, d) * e.sj[j];
    T *= d;
  }
  return q;
}

// The same from quad_edges_far's interval lengths
template <int NQ>
__device__ __forceinline__ float quad_sum(const QEdges<NQ>& e) {
  float q = 0.f;
  float T = __expf(-e.tau[0]);  // transmittance at edge j, carried along the edges
#pragma unroll
  for (int j = 0; j + 1 < NQ; ++j) {
    const float x = e.tau[j + 1] - e.tau[j];
    const float d = __expf(-x);
    q += T * e.delta[j] * phi_fn(x, d) * e.sj[j];
    T *= d;
  }
  return q;
}

// Consistency penalty of one Gaussian (App. E, regularisation): over each
// quadrature interval the reconstructed optical depth may not grow by less
// than the particle's own depth there, tau_ij = omega Sigma sqrt(pi/2)
// (erfc(b_j) - erfc(b_{j+1})), b = (t - mu) / (sqrt2 Sigma); for an edge left
// of the near bound b is taken at t_n, otherwise it is kappa x_j / sqrt2.
// P_i = sum_j max(0, tau_ij - (tau_{j+1} - tau_j))^2.
template <int NQ>
__device__ __forceinline__ float pair_penalty(const RayG& g, float tn, const QEdges<NQ>& e, const RenderArgs& a) {
  bool any_cl = false;
#pragma unroll
  for (int j = 0; j < NQ; ++j) any_cl = any_cl || e.cl[j];
  const float en = any_cl ? erfc_fast((tn - g.mu) * kInvSqrt2 * fast_rcp(g.sig)) : 0.f;
  const float cs = g.omega * g.sig * kSqrtHalfPi;
  float pen = 0.f;
#pragma unroll
  for (int j = 0; j + 1 < NQ; ++j) {
    const float e0 = e.cl[j] ? en : a.ecq[j];
    const float e1 = e.cl[j + 1] ? en : a.ecq[j + 1];
    const float r = fmaxf(cs * (e0 - e1) - (e.tau[j + 1] - e.tau[j]), 0.f);
    pen += r * r;
  }
  return pen;
}

// Quadrature of Eq. 7 for one Gaussian against the pixel's moment bounds.
template <int NH, int NQ>
__device__ __forceinline__ float particle_quadrature(const RayG& g, const PixelBasis& pb, const LInv<NH>& L,
                                                     float m0, float tn, const RenderArgs& a, QEdges<NQ>& e) {
  if constexpr (NH == 2)
    quad_edges_far<NQ>(g, pb, tn, a, e);
  else
    quad_edges<NQ>(g, pb, tn, a, e);
#pragma unroll
  for (int j = 0; j < NQ; ++j) e.tau[j] = m0 * bound_F<NH>(L, e.y[j], a.beta);
  if constexpr (NH == 2)
    return quad_sum<NQ>(e);
  else
    return quad_sum<NQ>(g, tn, e);
}

}  // namespace mb
