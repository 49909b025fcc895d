// Device-wide exclusive scan and a stable LSD radix sort used to build the
// per-tile Gaussian lists. No depth sort is needed: the moment and quadrature
// passes are order independent (Sec. 3.3), so lists are ordered by tile only,
// and by entry index inside a tile (stable), which keeps results bitwise
// reproducible.
#include "kernels.h"

namespace mb {

constexpr int kItems = 8;                  // items per thread
constexpr int kChunk = kBlock * kItems;    // items per block

__device__ __forceinline__ int wave_inclusive_sum(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    int u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// exclusive prefix of v over the 256 threads of the block; *total gets the sum
__device__ __forceinline__ int block_exclusive_sum(int v, int* lds4, int* total) {
  int inc = wave_inclusive_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 63) lds4[wave] = inc;
  __syncthreads();
  int off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    int s = lds4[w];
    off += (w < wave) ? s : 0;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return off + inc - v;
}

__global__ __launch_bounds__(256) void k_scan_reduce(const int* in, int64_t n, int* sums) {
  int64_t base = (int64_t)blockIdx.x * kChunk + threadIdx.x * kItems;
  int s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    int64_t i = base + k;
    s += (i < n) ? in[i] : 0;
  }
  __shared__ int lds[4];
  int tot;
  block_exclusive_sum(s, lds, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// single block: exclusive scan of `sums[0..m)` in place, total to *total
__global__ __launch_bounds__(256) void k_scan_top(int* sums, int64_t m, int* total) {
  int64_t per = (m + kBlock - 1) / kBlock;
  int64_t b0 = threadIdx.x * per;
  int s = 0;
  for (int64_t k = 0; k < per; ++k) {
    int64_t i = b0 + k;
    if (i < m) s += sums[i];
  }
  __shared__ int lds[4];
  int tot;
  int off = block_exclusive_sum(s, lds, &tot);
  for (int64_t k = 0; k < per; ++k) {
    int64_t i = b0 + k;
    if (i < m) {
      int v = sums[i];
      sums[i] = off;
      off += v;
    }
  }
  if (threadIdx.x == 0 && total != nullptr) *total = tot;
}

__global__ __launch_bounds__(256) void k_scan_down(const int* in, int* out, int64_t n, const int* sums) {
  int64_t base = (int64_t)blockIdx.x * kChunk + threadIdx.x * kItems;
  int v[kItems];
  int s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    int64_t i = base + k;
    v[k] = (i < n) ? in[i] : 0;
    s += v[k];
  }
  __shared__ int lds[4];
  int tot;
  int off = block_exclusive_sum(s, lds, &tot) + sums[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    int64_t i = base + k;
    if (i < n) out[i] = off;
    off += v[k];
  }
}

// Down-sweep that forms its block's offset itself: the sum of the block sums
// before it (fixed order), for at most kDirectBlocks blocks; block 0 also
// writes the total. Saves the single-block pass between the two sweeps.
constexpr int kDirectBlocks = 1024;

__global__ __launch_bounds__(256) void k_scan_down_direct(const int* in, int* out, int64_t n, const int* sums,
                                                          int nb, int* total) {
  __shared__ int lds[4];
  const int upto = total != nullptr && blockIdx.x == 0 ? nb : (int)blockIdx.x;
  int s = 0;
  for (int i = threadIdx.x; i < upto; i += kBlock) s += sums[i];
  int tot;
  block_exclusive_sum(s, lds, &tot);
  int before = tot;  // blocks [0, upto)
  if (blockIdx.x == 0) {
    if (total != nullptr && threadIdx.x == 0) *total = tot;
    before = 0;
  }
  int64_t base = (int64_t)blockIdx.x * kChunk + threadIdx.x * kItems;
  int v[kItems];
  int t = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    int64_t i = base + k;
    v[k] = (i < n) ? in[i] : 0;
    t += v[k];
  }
  int off = block_exclusive_sum(t, lds, &tot) + before;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    int64_t i = base + k;
    if (i < n) out[i] = off;
    off += v[k];
  }
}

// A kernel, not hipMemsetAsync: callers may capture the frame, and a graph's memset
// nodes have not been reliable on replays.
__global__ void k_zero_words(uint32_t* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

hipError_t launch_zero_words(void* p, int n, hipStream_t s) {
  if (n > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, (uint32_t*)p, n);
  return hipGetLastError();
}

size_t scan_tmp_ints(int64_t n) { return (size_t)((n + kChunk - 1) / kChunk) + 1; }

hipError_t launch_scan(const int* in, int* out, int64_t n, int* tmp, int* total, hipStream_t s) {
  int64_t nb = (n + kChunk - 1) / kChunk;
  if (nb == 0) {
    if (total) return launch_zero_words(total, 1, s);
    return hipSuccess;
  }
  hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kBlock), 0, s, in, n, tmp);
  if (nb <= kDirectBlocks) {
    hipLaunchKernelGGL(k_scan_down_direct, dim3((unsigned)nb), dim3(kBlock), 0, s, in, out, n, tmp, (int)nb,
                       total);
  } else {
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kBlock), 0, s, tmp, nb, total);
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kBlock), 0, s, in, out, n, tmp);
  }
  return hipGetLastError();
}

// Item count of a launch sized for n_max items: *n_dev when the count lives
// on the device (clamped to n_max), else n_max.
__device__ __forceinline__ int64_t items_of(const int* n_dev, int64_t n_max) {
  return n_dev ? min((int64_t)max(*n_dev, 0), n_max) : n_max;
}

// ---------------------------------------------------------------------------
// Radix sort, 8-bit digits. Per pass: block histograms (digit-major), the scan of
// their rows, then a stable scatter: every wave ranks a run of consecutive items
// with ballots, and the waves' counts give the block's order.
// ---------------------------------------------------------------------------
constexpr int kSortWaves = 8, kSortRounds = 8;
constexpr int kSortThreads = 64 * kSortWaves, kSortChunk = kSortThreads * kSortRounds;  // items per block

__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint32_t* keys, int64_t n_max, const int* n_dev,
                                                             int shift, int* hist, int nblocks) {
  const int64_t n = items_of(n_dev, n_max);
  __shared__ int h[256];
  if (threadIdx.x < 256) h[threadIdx.x] = 0;
  __syncthreads();
  int64_t base = (int64_t)blockIdx.x * kSortChunk;
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    int64_t i = base + r * kSortThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255u], 1);
  }
  __syncthreads();
  if (threadIdx.x < 256) hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// Ranks of a wave's run of items [i0, n), 64 a round, among the earlier items of
// the run with the same digit: place[r] = digit << 16 | rank of item i0 + 64 r +
// lane (all ones without one), cnt[d] the run's count of digit d.
template <int ROUNDS, class Digit>
__device__ __forceinline__ void rank_digits(int64_t i0, int64_t n, int* cnt, uint32_t* place, Digit&& digit) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt = (1ull << lane) - 1;
  for (int d = lane; d < 256; d += 64) cnt[d] = 0;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t i = i0 + 64 * r + lane;
    place[r] = ~0u;
    if (i0 + 64 * r >= n) continue;  // wave-uniform
    const bool valid = i < n;
    const uint32_t d = valid ? digit(r, i) : 0u;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const bool b = (d >> bit) & 1u;
      const uint64_t m = __ballot(b);
      peers &= b ? m : ~m;
    }
    const int rank = __popcll(peers & lt);
    const int before = valid ? cnt[d] : 0;
    __builtin_amdgcn_wave_barrier();
    if (valid && rank == 0) cnt[d] = before + __popcll(peers);
    __builtin_amdgcn_wave_barrier();
    if (valid) place[r] = (d << 16) | (uint32_t)(before + rank);
  }
}

// The block's items are put in digit order in LDS first, so that the stores run
// over consecutive addresses (16 items a run on average). Bound by the stores'
// lines: 12.8 us for 1.1 M entries, where 2048 items a block stored straight from
// the ranking took 17 to 19 us.
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(const uint32_t* keys_in, const int* vals_in,
                                                                uint32_t* keys_out, int* vals_out, int64_t n_max,
                                                                const int* n_dev, int shift, const int* hist,
                                                                int nblocks) {
  const int64_t n = items_of(n_dev, n_max);
  const int64_t base = (int64_t)blockIdx.x * kSortChunk;
  if (base >= n) return;
  __shared__ int cnt[kSortWaves][256];
  __shared__ int to[256];  // global minus local position of digit d's items
  __shared__ int lds[2][4];
  __shared__ uint32_t skey[kSortChunk];
  __shared__ int sval[kSortChunk];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t i0 = base + (int64_t)wave * 64 * kSortRounds;
  uint32_t key[kSortRounds], place[kSortRounds];
  int val[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int64_t i = i0 + 64 * r + lane;
    key[r] = i < n ? keys_in[i] : 0u;
    val[r] = i < n ? (vals_in ? vals_in[i] : (int)i) : 0;  // no vals_in: the identity
  }
  int total = 0, before = 0;  // of digit tid: all items, and those of the blocks before
  if (tid < 256) {
    const int* row = hist + (int64_t)tid * nblocks;  // inclusive counts
    total = row[nblocks - 1];
    before = blockIdx.x > 0 ? row[blockIdx.x - 1] : 0;
  }
  rank_digits<kSortRounds>(i0, n, cnt[wave], place,
                           [&](int r, int64_t) __attribute__((always_inline)) { return (key[r] >> shift) & 255u; });
  __syncthreads();
  int mine = 0;
  if (tid < 256)
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) mine += cnt[w][tid];
  const int gsum = wave_inclusive_sum(total), lsum = wave_inclusive_sum(mine);
  if (tid < 256 && lane == 63) {
    lds[0][wave] = gsum;
    lds[1][wave] = lsum;
  }
  __syncthreads();
  if (tid < 256) {
    int g = gsum - total + before, l = lsum - mine;
    for (int w = 0; w < wave; ++w) {
      g += lds[0][w];
      l += lds[1][w];
    }
    to[tid] = g - l;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      const int c = cnt[w][tid];
      cnt[w][tid] = l;
      l += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r)
    if (i0 + 64 * r + lane < n) {
      const int pos = cnt[wave][place[r] >> 16] + (int)(place[r] & 0xffffu);
      skey[pos] = key[r];
      sval[pos] = val[r];
    }
  __syncthreads();
  const int m = (int)min((int64_t)kSortChunk, n - base);
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int i = r * kSortThreads + tid;
    if (i < m) {
      const uint32_t k = skey[i];
      const int pos = to[(k >> shift) & 255u] + i;
      keys_out[pos] = k;
      vals_out[pos] = sval[i];
    }
  }
}

// In-place inclusive scan of the digit rows of the histogram (one block a row of
// nblocks counts); the digits' own offsets are the last counts of the rows before,
// which every scatter block adds up by itself.
__global__ __launch_bounds__(256) void k_radix_rows(int* hist, int nblocks) {
  __shared__ int lds[4];
  int* row = hist + (int64_t)blockIdx.x * nblocks;
  int before = 0;
  for (int b0 = 0; b0 < nblocks; b0 += kChunk) {
    const int base = b0 + threadIdx.x * kItems;
    int v[kItems], t = 0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      v[k] = base + k < nblocks ? row[base + k] : 0;
      t += v[k];
    }
    int tot;
    int off = block_exclusive_sum(t, lds, &tot) + before;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      off += v[k];
      if (base + k < nblocks) row[base + k] = off;
    }
    before += tot;
  }
}

size_t radix_tmp_ints(int64_t n) { return 256 * (size_t)((n + kSortChunk - 1) / kSortChunk) + 1; }

// one stable pass on digit (key >> shift) & 255
static hipError_t radix_pass(const uint32_t* kin, const int* vin, uint32_t* kout, int* vout, int64_t n,
                             const int* n_dev, int shift, int* tmp, hipStream_t s) {
  const int64_t nb = (n + kSortChunk - 1) / kSortChunk;
  int* hist = tmp;
  const dim3 grid((unsigned)nb), block(kSortThreads);
  hipLaunchKernelGGL(k_radix_hist, grid, block, 0, s, kin, n, n_dev, shift, hist, (int)nb);
  hipLaunchKernelGGL(k_radix_rows, dim3(256), dim3(kBlock), 0, s, hist, (int)nb);
  hipLaunchKernelGGL(k_radix_scatter, grid, block, 0, s, kin, vin, kout, vout, n, n_dev, shift, hist, (int)nb);
  return hipGetLastError();
}

int radix_passes(int bits) { return (bits + 7) / 8; }

hipError_t launch_radix_sort(uint32_t* const* keys, int* const* vals, int64_t n, const int* n_dev, int bits, int* tmp,
                             hipStream_t s) {
  const int passes = radix_passes(bits);
  if (n <= 0) return hipSuccess;
  for (int p = 0; p < passes; ++p) {
    const int in = (passes - p) & 1;  // the last pass writes buffer 0
    hipError_t e = radix_pass(keys[in], p == 0 ? nullptr : vals[in], keys[in ^ 1], vals[in ^ 1], n, n_dev, 8 * p, tmp,
                              s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_fill_ranges(int2* ranges, int n_keys) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n_keys) ranges[i] = make_int2(0, 0);
}

__global__ __launch_bounds__(256) void k_finish(const uint32_t* keys, const int* vals, const int* entry_rec,
                                                int64_t n_max, const int* n_dev, int* sorted_rec, int2* ranges) {
  const int64_t n = items_of(n_dev, n_max);
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int v = vals[i];
  sorted_rec[i] = entry_rec[v];
  uint32_t key = keys[i];
  if (i == 0 || keys[i - 1] != key) ranges[key].x = (int)i;
  if (i == n - 1 || keys[i + 1] != key) ranges[key].y = (int)(i + 1);
}

// Dispatch order of the tiles: heavy tiles (list longer than `split`) first,
// then the rest, each group longest first to a quantised length (one 8-bit
// radix pass; the sort is stable, so ties keep tile order). Heavy tiles start
// early instead of forming the tail of the launch, and consecutive blocks,
// which the hardware deals round-robin to the XCDs, spread them over all of
// them. Keys below 128 are exactly the heavy tiles.
__device__ __forceinline__ uint32_t tile_key(int len, int split) {
  return len > split ? 127u - (uint32_t)min((len - split - 1) >> 5, 127)  // 32 entries a step
                     : 255u - (uint32_t)min(len >> 2, 127);                // 4 entries a step
}
__global__ __launch_bounds__(256) void k_tile_keys(const int2* ranges, int n_keys, int split, uint32_t* keys,
                                                   int* vals) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_keys) return;
  int2 r = ranges[i];
  keys[i] = tile_key(max(r.y - r.x, 0), split);
  vals[i] = i;
}

// Block list of the render kernels from the ordered tiles: the first ns tiles
// (the heavy ones) get four blocks each, coded -(4 key + quadrant) - 1, then
// one block per remaining tile (its key), then blocks coded n_keys + ns that exit
// at once (the grid is render_blocks()).
__global__ __launch_bounds__(256) void k_block_list(const uint32_t* sorted_keys, const int* order, int n_keys,
                                                   int* blocks) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int total = render_blocks(n_keys);
  if (t >= total) return;
  // ns = number of leading tiles with a key below 128
  int lo = 0, hi = n_keys;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (sorted_keys[mid] < 128u) lo = mid + 1; else hi = mid;
  }
  const int ns = lo;
  if (t < n_keys) {
    if (t < ns) {
#pragma unroll
      for (int q = 0; q < 4; ++q) blocks[4 * t + q] = -(4 * order[t] + q) - 1;
    } else {
      blocks[3 * ns + t] = order[t];
    }
  } else if (t >= n_keys + 3 * ns) {
    blocks[t] = n_keys + ns;
  }
}

// ---------------------------------------------------------------------------
// Lists of few entries, and orders of few tiles, in one block: a launch costs more
// than the work of a pass over them, and each radix pass takes three.
// ---------------------------------------------------------------------------
constexpr int kSoloWaves = 16;

// Stable counting pass by digit (< 256) of the items [0, n), n <= kSoloItems, by
// all waves of the block: out(i, pos) for every item. Each wave takes a run of
// consecutive items. On return first[d] is the position of digit d's first item.
constexpr int kSoloRounds = 16, kSoloItems = 64 * kSoloWaves * kSoloRounds;
template <class Digit, class Out>
__device__ __forceinline__ void solo_pass(int n, int (*cnt)[256], int* first, int* lds4, Digit&& digit, Out&& out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int run = (n + 64 * kSoloWaves - 1) / (64 * kSoloWaves) * 64;
  const int i0 = wave * run, i1 = min(i0 + run, n);
  uint32_t place[kSoloRounds];
  rank_digits<kSoloRounds>(i0, i1, cnt[wave], place,
                           [&](int, int64_t i) __attribute__((always_inline)) { return digit((int)i); });
  __syncthreads();
  int c[kSoloWaves], tot = 0;
  if (tid < 256) {
#pragma unroll
    for (int w = 0; w < kSoloWaves; ++w) {
      c[w] = cnt[w][tid];
      tot += c[w];
    }
  }
  const int inc = wave_inclusive_sum(tot);
  if (tid < 256 && lane == 63) lds4[wave] = inc;
  __syncthreads();
  if (tid < 256) {
    int off = inc - tot;
    for (int w = 0; w < wave; ++w) off += lds4[w];
    first[tid] = off;
#pragma unroll
    for (int w = 0; w < kSoloWaves; ++w) {
      cnt[w][tid] = off;
      off += c[w];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSoloRounds; ++r) {
    const int i = i0 + 64 * r + lane;
    if (i < i1) out(i, cnt[wave][place[r] >> 16] + (int)(place[r] & 0xffffu));
  }
  __syncthreads();
}

// load(i) for the items [0, n), then store(i, value), by the whole block: eight
// loads of a thread in flight, for one block has nothing else to hide them behind
template <class Load, class Store>
__device__ __forceinline__ void solo_copy(int n, Load&& load, Store&& store) {
  constexpr int kThreads = 64 * kSoloWaves, kFlight = 8;
  for (int i0 = threadIdx.x; i0 < n; i0 += kFlight * kThreads) {
    decltype(load(0)) v[kFlight];
#pragma unroll
    for (int k = 0; k < kFlight; ++k) v[k] = load(min(i0 + k * kThreads, n - 1));
#pragma unroll
    for (int k = 0; k < kFlight; ++k)
      if (i0 + k * kThreads < n) store(i0 + k * kThreads, v[k]);
  }
}

// the block list (see k_block_list) from tile t's order, by the whole block
template <class Order>
__device__ __forceinline__ void write_block_list(int n_keys, int ns, int* blocks, Order&& order) {
  for (int t = threadIdx.x; t < render_blocks(n_keys); t += blockDim.x) {
    if (t < n_keys) {
      const int key = order(t);
      if (t < ns) {
#pragma unroll
        for (int q = 0; q < 4; ++q) blocks[4 * t + q] = -(4 * key + q) - 1;
      } else {
        blocks[3 * ns + t] = key;
      }
    } else if (t >= n_keys + 3 * ns) {
      blocks[t] = n_keys + ns;
    }
  }
}

// k_tile_keys, the sort and k_block_list in one block for at most kSoloItems
// tiles, which 14 bits of LDS order hold: 14 us for the 8160 tiles of 1920x1080, 8
// us for the 3024 of 1003x757, where the six launches take 25 and 20 us.
__global__ __launch_bounds__(64 * kSoloWaves) void k_solo_order(const int2* ranges, int n_keys, int split,
                                                                int* blocks) {
  __shared__ int cnt[kSoloWaves][256];
  __shared__ int first[256];
  __shared__ int lds4[4];
  __shared__ uint8_t keys[kSoloItems];
  __shared__ uint16_t order[kSoloItems];
  solo_copy(
      n_keys, [&](int i) __attribute__((always_inline)) { return ranges[i]; },
      [&](int i, int2 r) __attribute__((always_inline)) { keys[i] = (uint8_t)tile_key(max(r.y - r.x, 0), split); });
  __syncthreads();
  solo_pass(
      n_keys, cnt, first, lds4, [&](int i) __attribute__((always_inline)) { return (uint32_t)keys[i]; },
      [&](int i, int pos) __attribute__((always_inline)) { order[pos] = (uint16_t)i; });
  write_block_list(n_keys, first[128], blocks, [&](int t) __attribute__((always_inline)) { return (int)order[t]; });
}

// The sort of the emitted entries, the per-tile ranges and the block list in one
// block for a list (or, with the count on the device, a capacity) of at most
// kSoloItems entries and kSoloKeys tiles, as much as two buffers and the ranges
// fill the LDS with: 16 us for 5500 entries on 64 tiles, where the eight launches
// of the general path take 31 us. At the limits the two are alike.
constexpr int kSoloKeys = 2048;
__global__ __launch_bounds__(64 * kSoloWaves) void k_solo_lists(const uint32_t* keys, const int* entry_rec, int n_max,
                                                                const int* n_dev, int n_keys, int passes, int split,
                                                                int* vals, int* sorted_rec, int2* ranges,
                                                                int* blocks) {
  const int n = (int)items_of(n_dev, n_max);
  __shared__ int cnt[kSoloWaves][256];
  __shared__ int first[256];
  __shared__ int lds4[4];
  __shared__ uint32_t buf[2][kSoloItems];  // key << 16 | entry
  __shared__ uint16_t beg[kSoloKeys], end[kSoloKeys];
  solo_copy(
      n, [&](int i) __attribute__((always_inline)) { return keys[i]; },
      [&](int i, uint32_t key) __attribute__((always_inline)) { buf[0][i] = (key << 16) | (uint32_t)i; });
  for (int t = threadIdx.x; t < n_keys; t += blockDim.x) beg[t] = end[t] = 0;
  __syncthreads();
  for (int p = 0; p < passes; ++p) {
    const uint32_t* in = buf[p & 1];
    uint32_t* to = buf[(p & 1) ^ 1];
    solo_pass(
        n, cnt, first, lds4, [&](int i) __attribute__((always_inline)) { return (in[i] >> (16 + 8 * p)) & 255u; },
        [&](int i, int pos) __attribute__((always_inline)) { to[pos] = in[i]; });
  }
  const uint32_t* sorted = buf[passes & 1];
  solo_copy(
      n, [&](int i) __attribute__((always_inline)) { return entry_rec[sorted[i] & 0xffffu]; },
      [&](int i, int rec) __attribute__((always_inline)) {
        const uint32_t e = sorted[i], key = e >> 16;
        vals[i] = (int)(e & 0xffffu);
        sorted_rec[i] = rec;
        if (i == 0 || (sorted[i - 1] >> 16) != key) beg[key] = (uint16_t)i;
        if (i == n - 1 || (sorted[i + 1] >> 16) != key) end[key] = (uint16_t)(i + 1);
      });
  __syncthreads();
  uint32_t* order = buf[(passes & 1) ^ 1];
  for (int t = threadIdx.x; t < n_keys; t += blockDim.x) ranges[t] = make_int2(beg[t], end[t]);
  solo_pass(
      n_keys, cnt, first, lds4,
      [&](int i) __attribute__((always_inline)) { return tile_key((int)end[i] - (int)beg[i], split); },
      [&](int i, int pos) __attribute__((always_inline)) { order[pos] = (uint32_t)i; });
  write_block_list(n_keys, first[128], blocks, [&](int t) __attribute__((always_inline)) { return (int)order[t]; });
}

bool solo_lists(int64_t n, int n_keys) { return n > 0 && n <= kSoloItems && n_keys <= kSoloKeys; }

hipError_t launch_solo_lists(const uint32_t* keys, const int* entry_rec, int64_t n, const int* n_dev, int n_keys,
                             int bits, int split, int* vals, int* sorted_rec, int2* ranges, int* blocks, hipStream_t s) {
  hipLaunchKernelGGL(k_solo_lists, dim3(1), dim3(64 * kSoloWaves), 0, s, keys, entry_rec, (int)n, n_dev, n_keys,
                     radix_passes(bits), split, vals, sorted_rec, ranges, blocks);
  return hipGetLastError();
}

size_t order_tmp_ints(int n_keys) { return 4 * (size_t)n_keys + radix_tmp_ints(n_keys); }

hipError_t launch_tile_order(const int2* ranges, int n_keys, int split, int* blocks, int* tmp, hipStream_t s) {
  if (n_keys <= 0) return hipSuccess;
  if (n_keys <= kSoloItems) {
    hipLaunchKernelGGL(k_solo_order, dim3(1), dim3(64 * kSoloWaves), 0, s, ranges, n_keys, split, blocks);
    return hipGetLastError();
  }
  uint32_t* ka = reinterpret_cast<uint32_t*>(tmp);
  uint32_t* kb = ka + n_keys;
  int* va = tmp + 2 * (size_t)n_keys;
  int* vb = tmp + 3 * (size_t)n_keys;
  int* rt = tmp + 4 * (size_t)n_keys;
  hipLaunchKernelGGL(k_tile_keys, dim3((n_keys + 255) / 256), dim3(256), 0, s, ranges, n_keys, split, ka, va);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = radix_pass(ka, va, kb, vb, n_keys, nullptr, 0, rt, s);
  if (e != hipSuccess) return e;
  int total = render_blocks(n_keys);
  hipLaunchKernelGGL(k_block_list, dim3((total + 255) / 256), dim3(256), 0, s, kb, vb, n_keys, blocks);
  return hipGetLastError();
}

hipError_t launch_finish_lists(const uint32_t* keys, const int* vals, const int* entry_rec, int64_t n,
                               const int* n_dev, int* sorted_rec, int2* ranges, int n_keys, bool ranges_cleared,
                               hipStream_t s) {
  if (!ranges_cleared)
    hipLaunchKernelGGL(k_fill_ranges, dim3((n_keys + 255) / 256), dim3(256), 0, s, ranges, n_keys);
  if (n > 0)
    hipLaunchKernelGGL(k_finish, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, keys, vals, entry_rec,
                       n, n_dev, sorted_rec, ranges);
  return hipGetLastError();
}

}  // namespace mb
