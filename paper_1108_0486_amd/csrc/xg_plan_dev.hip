// Device-side batch planner of libxg: turns a request table in the caller's
// array order into the table the persistent batch kernels serve.  Requests of
// one stream become one group, kept in array order (that is what makes a
// batched request read the positions it would read alone); a group of one
// long request may become tiles of L words that separate wavefronts run from
// jumped start states (Section 2: independent subsequences of one stream);
// queue items are ordered largest first, so the dynamic queue balances uneven
// lengths.  Everything runs as kernels on the caller's stream, so the call
// needs no host round trip and can be captured in a HIP graph.
//
// Grouping is a sort of 64-bit keys (stream << 32 | request index): the keys
// are distinct, so any correct sort leaves each stream's requests in array
// order.  The queue items are sorted the same way on (inverted cost << 32 |
// group << 8 | tile).  Launches bound a plan of ordinary size (3 to 8 us each,
// most of it not work), so each step does all it can before it needs the whole
// table again: a sort is one launch over blocks of 1024 keys and one for each
// eightfold merge, and the producer of a prefix sum's input leaves its block sums.
// Without tiles a plan takes 10 launches up to 16384 requests, 12 at 65536 and 16 at
// a million (two more with tiles); it took 28 at 8192, 32 at 16384, 44 at 65536 and 74.
// Plan and batch of short requests: 4100 requests 126 -> 65 us, 16384 199 -> 126,
// 65536 281 -> 173, 900000 1130 -> 952.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xg_device.h"
#include "xg_host.h"
#include "xg_internal.h"
#include "xg_launch.h"
#include "xg_plan_dev.h"

namespace xg {
namespace {

constexpr uint32_t kSortBlock = 1024;    // keys one workgroup sorts (kSortThreads threads, two each)
constexpr uint32_t kSortThreads = 512;
constexpr uint32_t kLeastKeys = 2048;    // keys that a table has room for at least
constexpr uint32_t kScanBlock = 1024;  // elements one scan workgroup covers (256 threads, four each)

// Planner counters (meta words).
constexpr uint32_t kMetaValid = 0;  // requests that passed the checks
constexpr uint32_t kMetaTiles = 1;  // tile slots used (the largest tile prefix sum within max_tiles)
constexpr uint32_t kMetaItems = 2;  // queue items

__device__ __forceinline__ uint64_t words_of(uint64_t n, uint32_t dtype) {
  return dtype == XG_NORMAL ? n + (n & 1u) : n;
}

// Cost of serving n values of dtype in the queue's balance (the host
// planner's measure: words consumed, normals weighted four times for their
// transcendental work).
__device__ __forceinline__ uint64_t cost_of(uint64_t n, uint32_t dtype) {
  return dtype == XG_NORMAL ? 4u * words_of(n, dtype) : n;
}

// Queue item key: larger cost sorts first, then group, then tile.
__device__ __forceinline__ uint64_t item_key(uint64_t cost, uint32_t g, uint32_t k) {
  const uint32_t c = cost > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)cost;
  return ((uint64_t)(0xFFFFFFFFu - c) << 32) | ((uint64_t)g << 8) | k;
}

// ---- sums and sorts inside a workgroup ---------------------------------------

// The sum of every thread's v.  wsum holds a value per wavefront.
template <typename T, uint32_t THREADS>
__device__ __forceinline__ T wg_sum(T v, T *wsum) {
#pragma unroll
  for (uint32_t d = 32; d; d >>= 1) v += __shfl_xor(v, d);
  if ((threadIdx.x & 63u) == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  T all = 0;
#pragma unroll
  for (uint32_t i = 0; i < THREADS / 64; ++i) all += wsum[i];
  __syncthreads();  // wsum may be reused after this
  return all;
}

// Exclusive prefix sums of the workgroup's values, EPT consecutive ones per
// thread (v[e] is element EPT t + e): on return v[e] holds the sum of every
// element before it, and *total the sum of all.  wsum holds a value per wavefront.
template <typename T, uint32_t THREADS, uint32_t EPT>
__device__ __forceinline__ void wg_exclusive(T (&v)[EPT], T *wsum, T *total) {
  constexpr uint32_t kWaves = THREADS / 64;
  const uint32_t t = threadIdx.x, lane = t & 63u, w = t >> 6;
  T mine = 0;
#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) mine += v[e];
  T x = mine;
#pragma unroll
  for (uint32_t d = 1; d < 64u; d <<= 1) {
    const T y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63u) wsum[w] = x;
  __syncthreads();
  T run = x - mine, all = 0;
#pragma unroll
  for (uint32_t i = 0; i < kWaves; ++i) {
    const T s = wsum[i];
    if (i < w) run += s;
    all += s;
  }
  *total = all;
  __syncthreads();  // wsum is reused by the next scan
#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) {
    const T here = v[e];
    v[e] = run;
    run += here;
  }
}

// One compare-exchange pass (stage K, distance J) of the bitonic network on
// element EPT t + e in k[e].  Distances of a wavefront or more go through one
// half of lds (2 N keys), the halves in turn, so that one barrier is enough.
template <uint32_t N, uint32_t THREADS, uint32_t K, uint32_t J>
__device__ __forceinline__ void sort_pass(uint64_t (&k)[N / THREADS], uint64_t *lds, uint32_t &half) {
  constexpr uint32_t EPT = N / THREADS;
  const uint32_t i0 = threadIdx.x * EPT;
  if constexpr (J < EPT) {
#pragma unroll
    for (uint32_t e = 0; e < EPT; ++e) {
      if (e & J) continue;
      const bool asc = ((i0 + e) & K) == 0u;
      const uint64_t x = k[e], y = k[e | J];
      const bool swap = (x > y) == asc;
      k[e] = swap ? y : x;
      k[e | J] = swap ? x : y;
    }
  } else {
    uint64_t y[EPT];
    if constexpr (J < 64 * EPT) {
#pragma unroll
      for (uint32_t e = 0; e < EPT; ++e) y[e] = dev::lane_xor<J / EPT>(k[e]);
    } else {
      uint64_t *s = lds + half * N;
      half ^= 1u;
#pragma unroll
      for (uint32_t e = 0; e < EPT; ++e) s[i0 + e] = k[e];
      __syncthreads();
#pragma unroll
      for (uint32_t e = 0; e < EPT; ++e) y[e] = s[(i0 + e) ^ J];
    }
#pragma unroll
    for (uint32_t e = 0; e < EPT; ++e) {
      const uint32_t i = i0 + e;
      const bool least = ((i & J) == 0u) == ((i & K) == 0u);  // the lower place of an ascending pair, and so on
      k[e] = (k[e] > y[e]) == least ? y[e] : k[e];
    }
  }
}

template <uint32_t N, uint32_t THREADS, uint32_t K, uint32_t J>
__device__ __forceinline__ void sort_passes(uint64_t (&k)[N / THREADS], uint64_t *lds, uint32_t &half) {
  sort_pass<N, THREADS, K, J>(k, lds, half);
  if constexpr (J > 1) sort_passes<N, THREADS, K, J / 2>(k, lds, half);
}

// Sorts the workgroup's N distinct-or-all-ones keys ascending.  lds holds 2 N keys.
template <uint32_t N, uint32_t THREADS, uint32_t K = 2>
__device__ __forceinline__ void wg_sort(uint64_t (&k)[N / THREADS], uint64_t *lds, uint32_t &half) {
  sort_passes<N, THREADS, K, K / 2>(k, lds, half);
  if constexpr (K < N) wg_sort<N, THREADS, 2 * K>(k, lds, half);
}

// ---- sort of 64-bit keys over the device -------------------------------------

// Sorts each kSortBlock places of a table of keys, src to dst (which may be the
// same).  REQS: key i is request i's (stream << 32 | i), with stream 0xFFFFFFFF
// (sorted after every valid stream) for a request that fails the checks and all
// ones past the table; the launch also clears the counters.
template <bool REQS>
__global__ __launch_bounds__(kSortThreads) void k_sort_blocks(const uint64_t *src, uint64_t *dst,
                                                      const xg_request *__restrict__ reqs, uint32_t num_reqs,
                                                      uint64_t num_streams, uint32_t *__restrict__ work,
                                                      uint32_t *__restrict__ meta) {
  __shared__ uint64_t lds[2 * kSortBlock];
  const uint32_t t = threadIdx.x, i0 = blockIdx.x * kSortBlock + 2u * t;
  uint64_t key[2];
  uint32_t half = 0;
#pragma unroll
  for (uint32_t e = 0; e < 2u; ++e) {
    if constexpr (REQS) {
      const uint32_t i = i0 + e;
      key[e] = ~0ull;
      if (i < num_reqs) {
        const xg_request q = reqs[i];
        const bool valid = q.stream < num_streams && q.dtype <= XG_NORMAL && q.flags == 0u;
        key[e] = ((valid ? q.stream : 0xFFFFFFFFull) << 32) | i;
      }
    } else {
      key[e] = src[i0 + e];
    }
  }
  if (REQS && blockIdx.x == 0 && t < 64u) {
    work[t] = 0u;
    meta[t] = 0u;
  }
  wg_sort<kSortBlock, kSortThreads>(key, lds, half);
#pragma unroll
  for (uint32_t e = 0; e < 2u; ++e) dst[i0 + e] = key[e];
}

// Merges each W sorted runs of 2^run_log2 keys of src into one of dst: a key's
// place is its own in its run plus, for each other run, the keys there that
// come before it (equal keys, the all-ones ones, in run order), found by W
// searches side by side.  The chain of a search's loads bounds it while the table is
// small (8192 keys of 1024 in 5.4 us, 16384 in 8 us; the bitonic passes that
// one merge stands for took seven launches, 35 us), the number of loads when it
// is large.
template <uint32_t W>
__global__ __launch_bounds__(256) void k_merge(const uint64_t *__restrict__ src, uint64_t *__restrict__ dst,
                                               uint32_t n, uint32_t run_log2) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  const uint32_t run = 1u << run_log2, base = i & ~(W * run - 1u);
  const uint32_t mine = (i - base) >> run_log2;
  const uint64_t x = src[i];
  uint32_t at[W];  // keys of run q known to come before x
#pragma unroll
  for (uint32_t q = 0; q < W; ++q) at[q] = 0;
  for (uint32_t step = run >> 1; step; step >>= 1) {
#pragma unroll
    for (uint32_t q = 0; q < W; ++q) {
      const uint64_t y = src[base + (q << run_log2) + at[q] + step - 1u];
      if (y < x || (y == x && q < mine)) at[q] += step;
    }
  }
  uint32_t place = base + (i & (run - 1u));
#pragma unroll
  for (uint32_t q = 0; q < W; ++q) {
    const uint64_t y = src[base + (q << run_log2) + at[q]];
    const uint32_t before = at[q] + (y < x || (y == x && q < mine) ? 1u : 0u);
    place += q == mine ? 0u : before;
  }
  dst[place] = x;
}

uint32_t log2_of(uint32_t pow2) { return 31u - (uint32_t)__builtin_clz(pow2); }

// Sorts a[0, n) ascending, n a power of two >= kSortBlock, with tmp for n keys;
// with reqs the keys are theirs (k_sort_blocks).  Merges are eightfold, or
// sixteenfold where one then ends the sort; wider ones search more than a pass
// saves (plan and batch of 900000 short requests: 952 us with eight, 1049 with
// sixteen).
hipError_t sort_keys(uint64_t *a, uint64_t *tmp, uint32_t n, const xg_request *reqs, uint32_t num_reqs,
                     uint64_t num_streams, uint32_t *work, uint32_t *meta, hipStream_t stream) {
  uint32_t run = log2_of(kSortBlock), left = log2_of(n) - run;  // merges left, in powers of two
  const uint32_t most = left == 4 ? 4 : 3, passes = (left + most - 1) / most;
  uint64_t *at = passes % 2 ? tmp : a;  // so that the last pass ends in a
  const dim3 blocks(n / kSortBlock), threads(kSortThreads);
  hipError_t e =
      reqs ? launch(k_sort_blocks<true>, blocks, threads, 0, stream, a, at, reqs, num_reqs, num_streams, work, meta)
           : launch(k_sort_blocks<false>, blocks, threads, 0, stream, a, at, reqs, num_reqs, num_streams, work, meta);
  while (left && e == hipSuccess) {
    uint64_t *to = at == a ? tmp : a;
    const dim3 grid((n + 255) / 256), b256(256);
    const uint32_t by = left < most ? left : most;
    e = by == 4   ? launch(k_merge<16>, grid, b256, 0, stream, at, to, n, run)
        : by == 3 ? launch(k_merge<8>, grid, b256, 0, stream, at, to, n, run)
        : by == 2 ? launch(k_merge<4>, grid, b256, 0, stream, at, to, n, run)
                  : launch(k_merge<2>, grid, b256, 0, stream, at, to, n, run);
    at = to;
    run += by;
    left -= by;
  }
  return e;
}

// ---- exclusive prefix sums in place, total at a[n] ---------------------------

// The kernel that writes a[0, n) leaves the sum of each kScanBlock values in
// sums, and the scan's workgroups add up the sums before their own (at most
// 1024 of them).
template <typename T>
__device__ __forceinline__ T sums_before(const T *__restrict__ sums, T *wsum) {
  T v = 0;
  for (uint32_t b = threadIdx.x; b < blockIdx.x; b += 256u) v += sums[b];
  return wg_sum<T, 256>(v, wsum);
}

// Exclusive prefix sums of this workgroup's kScanBlock values of a[0, n), four
// per thread, in x (0 past n) and in a; the last workgroup writes a[n].
template <typename T>
__device__ __forceinline__ void scan_block(T *__restrict__ a, uint32_t n, const T *__restrict__ sums, T (&x)[4],
                                           T *wsum) {
  const uint32_t i0 = blockIdx.x * kScanBlock + 4u * threadIdx.x;
#pragma unroll
  for (uint32_t q = 0; q < 4u; ++q) x[q] = i0 + q < n ? a[i0 + q] : T(0);
  const T base = sums_before(sums, wsum);
  T total;
  wg_exclusive<T, 256, 4>(x, wsum, &total);
#pragma unroll
  for (uint32_t q = 0; q < 4u; ++q) {
    x[q] += base;
    if (i0 + q < n) a[i0 + q] = x[q];
  }
  if (blockIdx.x == gridDim.x - 1u && threadIdx.x == 0) a[n] = base + total;
}

__global__ __launch_bounds__(256) void k_scan(uint32_t *__restrict__ a, uint32_t n,
                                              const uint32_t *__restrict__ sums) {
  __shared__ uint32_t wsum[4];
  uint32_t x[4];
  scan_block(a, n, sums, x, wsum);
}

// ---- planner steps -----------------------------------------------------------

// For sorted position i: heads[i] = 1 where a group starts, costs[i] = the
// request's cost (both 0 past the valid requests), and their sums by
// kScanBlock; the number of valid requests, and the error word where one is not.
__global__ __launch_bounds__(256) void k_plan_heads(const xg_request *__restrict__ reqs, uint32_t num_reqs,
                                                    const uint64_t *__restrict__ keys, uint32_t *__restrict__ meta,
                                                    uint32_t *__restrict__ work, uint32_t *__restrict__ heads,
                                                    uint64_t *__restrict__ costs, uint32_t *__restrict__ head_sums,
                                                    uint64_t *__restrict__ cost_sums) {
  __shared__ uint32_t wsum32[4];
  __shared__ uint64_t wsum[4];
  const uint32_t i0 = blockIdx.x * kScanBlock + 4u * threadIdx.x;
  uint32_t my_heads = 0;
  uint64_t my_costs = 0;
#pragma unroll
  for (uint32_t e = 0; e < 4u; ++e) {
    const uint32_t i = i0 + e;
    if (i >= num_reqs) continue;
    const uint64_t k = keys[i];
    uint32_t head = 0;
    uint64_t cost = 0;
    if ((k >> 32) != 0xFFFFFFFFull) {
      head = i == 0 || (k >> 32) != (keys[i - 1] >> 32);
      const xg_request q = reqs[(uint32_t)k];
      cost = cost_of(q.n, q.dtype);
      if (i + 1 == num_reqs || (keys[i + 1] >> 32) == 0xFFFFFFFFull) meta[kMetaValid] = i + 1;
    } else if (i + 1 == num_reqs) {
      work[1] = 1u;
    }
    heads[i] = head;
    costs[i] = cost;
    my_heads += head;
    my_costs += cost;
  }
  const uint32_t h = wg_sum<uint32_t, 256>(my_heads, wsum32);
  const uint64_t c = wg_sum<uint64_t, 256>(my_costs, wsum);
  if (threadIdx.x == 0) {
    head_sums[blockIdx.x] = h;
    cost_sums[blockIdx.x] = c;
  }
}

// Prefix sums of heads (each request's group) and costs; hp[g] = first sorted
// position of group g, and hp[G] = the number of valid requests; every tile
// prefix sum 0 where there are no tiles, and every queue item all ones.
__global__ __launch_bounds__(256) void k_plan_groups(uint32_t num_reqs, uint32_t *__restrict__ heads,
                                                     uint64_t *__restrict__ costs,
                                                     const uint32_t *__restrict__ head_sums,
                                                     const uint64_t *__restrict__ cost_sums,
                                                     const uint32_t *__restrict__ meta, uint32_t *__restrict__ hp,
                                                     uint32_t *__restrict__ zero_tiles,
                                                     uint64_t *__restrict__ items, uint32_t item_n) {
  __shared__ uint32_t wsum32[4];
  __shared__ uint64_t wsum[4];
  const uint32_t i0 = blockIdx.x * kScanBlock + 4u * threadIdx.x;
  bool head[4];
#pragma unroll
  for (uint32_t q = 0; q < 4u; ++q) head[q] = i0 + q < num_reqs && heads[i0 + q] != 0u;
  uint32_t g[4];
  uint64_t c[4];
  scan_block(heads, num_reqs, head_sums, g, wsum32);
  scan_block(costs, num_reqs, cost_sums, c, wsum);
#pragma unroll
  for (uint32_t q = 0; q < 4u; ++q)
    if (head[q]) hp[g[q]] = i0 + q;
  if (blockIdx.x == gridDim.x - 1u && threadIdx.x == 0) hp[heads[num_reqs]] = meta[kMetaValid];
  const uint32_t step = gridDim.x * 256u, t = blockIdx.x * 256u + threadIdx.x;
  if (zero_tiles)
    for (uint32_t i = t; i <= num_reqs; i += step) zero_tiles[i] = 0u;
  for (uint32_t i = t; i < item_n; i += step) items[i] = ~0ull;
}

// tiles[g] = the tiles group g asks for: ceil(words / L) for a group of one
// request split into 2 .. kMaxSegments tiles, else 0; and their sums.
__global__ __launch_bounds__(256) void k_plan_want(const xg_request *__restrict__ reqs, uint32_t num_reqs,
                                                   const uint64_t *__restrict__ keys,
                                                   const uint32_t *__restrict__ heads,
                                                   const uint32_t *__restrict__ hp, uint64_t tile_words,
                                                   uint32_t *__restrict__ tiles, uint32_t *__restrict__ sums) {
  __shared__ uint32_t wsum[4];
  const uint32_t g0 = blockIdx.x * kScanBlock + 4u * threadIdx.x, num_groups = heads[num_reqs];
  uint32_t mine = 0;
#pragma unroll
  for (uint32_t e = 0; e < 4u; ++e) {
    const uint32_t g = g0 + e;
    if (g >= num_reqs) continue;
    uint32_t want = 0;
    if (g < num_groups && hp[g + 1] - hp[g] == 1u) {
      const xg_request q = reqs[(uint32_t)keys[hp[g]]];
      const uint64_t parts = (words_of(q.n, q.dtype) + tile_words - 1) / tile_words;
      if (parts > 1 && parts <= kMaxSegments) want = (uint32_t)parts;
    }
    tiles[g] = want;
    mine += want;
  }
  const uint32_t all = wg_sum<uint32_t, 256>(mine, wsum);
  if (threadIdx.x == 0) sums[blockIdx.x] = all;
}

// Prefix sums of tiles.  Groups split in order while their tiles fit max_tiles
// slots; meta[kMetaTiles] = the slots so used.
__global__ __launch_bounds__(256) void k_plan_budget(uint32_t num_reqs, uint32_t *__restrict__ tiles,
                                                     const uint32_t *__restrict__ sums, uint32_t max_tiles,
                                                     uint32_t *__restrict__ meta) {
  __shared__ uint32_t wsum[4];
  const uint32_t i0 = blockIdx.x * kScanBlock + 4u * threadIdx.x;
  uint32_t x[4];
  scan_block(tiles, num_reqs, sums, x, wsum);
  uint32_t most = 0;
#pragma unroll
  for (uint32_t q = 0; q < 4u; ++q)
    if (i0 + q < num_reqs && x[q] <= max_tiles) most = x[q];
  if (blockIdx.x == gridDim.x - 1u && threadIdx.x == 0 && tiles[num_reqs] <= max_tiles) most = tiles[num_reqs];
#pragma unroll
  for (uint32_t d = 32; d; d >>= 1) {
    const uint32_t other = __shfl_xor(most, d);
    most = other > most ? other : most;
  }
  if ((threadIdx.x & 63u) == 0 && most) atomicMax(&meta[kMetaTiles], most);
}

__device__ __forceinline__ bool group_split(const uint32_t *tiles, uint32_t g, uint32_t used) {
  return tiles[g + 1] != tiles[g] && tiles[g + 1] <= used;
}

// Queue items: tile k of split group g at slot tiles[g] + k, every other group
// g at tile_cap + g (unused places keep all ones and sort last).
__global__ __launch_bounds__(256) void k_plan_items(const xg_request *__restrict__ reqs, uint32_t num_reqs,
                                                    const uint64_t *__restrict__ keys,
                                                    const uint32_t *__restrict__ heads,
                                                    const uint64_t *__restrict__ costs,
                                                    const uint32_t *__restrict__ hp,
                                                    const uint32_t *__restrict__ tiles, uint64_t tile_words,
                                                    uint32_t tile_cap, uint32_t *__restrict__ meta,
                                                    uint64_t *__restrict__ items) {
  const uint32_t g = blockIdx.x * 256u + threadIdx.x;
  if (g >= num_reqs || g >= heads[num_reqs]) return;
  if (group_split(tiles, g, meta[kMetaTiles])) {
    const xg_request q = reqs[(uint32_t)keys[hp[g]]];
    const uint32_t t = tiles[g + 1] - tiles[g];
    for (uint32_t k = 0; k < t; ++k) {
      const uint64_t first = k * tile_words;
      const uint64_t nk = q.n - first < tile_words ? q.n - first : tile_words;
      items[tiles[g] + k] = item_key(cost_of(nk, q.dtype), g, k);
    }
    atomicAdd(&meta[kMetaItems], t);
  } else {
    items[tile_cap + g] = item_key(costs[hp[g + 1]] - costs[hp[g]], g, 0);
    atomicAdd(&meta[kMetaItems], 1u);
  }
}

// offs[p] = table entries of sorted item p (0 past the items), and their sums.
__global__ __launch_bounds__(256) void k_plan_counts(uint32_t item_n, const uint64_t *__restrict__ items,
                                                     const uint32_t *__restrict__ hp,
                                                     const uint32_t *__restrict__ tiles,
                                                     const uint32_t *__restrict__ meta, uint32_t *__restrict__ offs,
                                                     uint32_t *__restrict__ sums) {
  __shared__ uint32_t wsum[4];
  const uint32_t p0 = blockIdx.x * kScanBlock + 4u * threadIdx.x;
  uint32_t mine = 0;
#pragma unroll
  for (uint32_t e = 0; e < 4u; ++e) {
    const uint32_t p = p0 + e;
    if (p >= item_n) continue;
    uint32_t cnt = 0;
    if (p < meta[kMetaItems]) {
      const uint32_t g = (uint32_t)items[p] >> 8;
      cnt = group_split(tiles, g, meta[kMetaTiles]) ? 1u : hp[g + 1] - hp[g];
    }
    offs[p] = cnt;
    mine += cnt;
  }
  const uint32_t all = wg_sum<uint32_t, 256>(mine, wsum);
  if (threadIdx.x == 0) sums[blockIdx.x] = all;
}

// Table entry e: the j-th request of its item's group, or the item's tile as a
// segment entry.  Entry 0 also publishes the counts for the batch kernel.
__global__ __launch_bounds__(256) void k_plan_emit(const xg_request *__restrict__ reqs,
                                                   const uint64_t *__restrict__ keys,
                                                   const uint32_t *__restrict__ hp,
                                                   const uint32_t *__restrict__ tiles, uint64_t tile_words,
                                                   const uint64_t *__restrict__ items, uint32_t item_n,
                                                   const uint32_t *__restrict__ offs,
                                                   const uint32_t *__restrict__ meta,
                                                   xg_request *__restrict__ table, uint32_t *__restrict__ work) {
  const uint32_t e = blockIdx.x * 256u + threadIdx.x;
  const uint32_t num_items = meta[kMetaItems], entries = offs[item_n];
  if (e == 0) {
    work[2] = num_items;
    work[3] = entries;
  }
  if (e >= entries) return;
  // The item holding entry e: the last p < num_items with offs[p] <= e.
  uint32_t lo = 0, hi = num_items;  // offs[lo] <= e < offs[hi]
  while (hi - lo > 1u) {
    const uint32_t mid = (lo + hi) >> 1;
    if (offs[mid] <= e) lo = mid;
    else hi = mid;
  }
  const uint64_t it = items[lo];
  const uint32_t g = (uint32_t)it >> 8, k = (uint32_t)it & 0xFFu;
  if (group_split(tiles, g, meta[kMetaTiles])) {
    xg_request q = reqs[(uint32_t)keys[hp[g]]];
    const uint64_t first = k * tile_words;
    const uint32_t t = tiles[g + 1] - tiles[g], slot = tiles[g] + k;
    q.n = q.n - first < tile_words ? q.n - first : tile_words;
    q.out_offset += first;
    q.flags = kReqSegment | (k << 8) | (slot << 16) | (k + 1 == t ? kReqLast : 0u);
    table[e] = q;
  } else {
    table[e] = reqs[(uint32_t)keys[hp[g] + (e - offs[lo])]];
  }
}

// ---- small tables: the whole plan in one workgroup ---------------------------

// Table entries plus tile slots that one workgroup plans with a single launch
// instead of the multi-kernel sequence above (the plan is the same): N
// elements, EPT = N / THREADS consecutive ones per thread, N from 256 to 4096 (160
// KB of LDS).  Latency bounds it, so the sorts keep their keys in registers
// and exchange them by lane swaps; only distances beyond a wavefront go
// through LDS, with one barrier each.  384 requests take 9 us (24 us with
// every pass through LDS in 1024 elements).
constexpr uint32_t kSmallPlanMax = 4096;

// Adds the workgroup's flags to *count: one atomic per wavefront.
template <uint32_t EPT>
__device__ __forceinline__ void count_flags(const bool (&f)[EPT], uint32_t *count) {
  uint32_t c = 0;
#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) c += (uint32_t)__popcll(__ballot(f[e]));
  if ((threadIdx.x & 63u) == 0 && c) atomicAdd(count, c);
}

// The planner for num_reqs + tile_cap <= N: the steps of the kernels above
// (keys, sort, group heads and cost sums, tiles and their budget, queue items,
// their sort, entry counts, table) on EPT consecutive elements per thread.
// Writes offs[0 .. num_reqs + tile_cap], the table and work[0 .. 63] (counts
// in work[2], work[3], the error word in work[1]).
template <uint32_t N, uint32_t THREADS>
__global__ __launch_bounds__(THREADS) void k_plan_small(const xg_request *__restrict__ reqs, uint32_t num_reqs,
                                                        uint64_t num_streams, uint64_t tile_words, uint32_t tile_cap,
                                                        uint32_t *__restrict__ work, uint32_t *__restrict__ offs_out,
                                                        xg_request *__restrict__ table) {
  constexpr uint32_t EPT = N / THREADS;
  __shared__ uint64_t swap[2 * N];   // the sorts' exchanges; between them the item keys by place
  __shared__ uint64_t costs[N + 1];  // request costs by index, then cost prefix sums over sorted requests
  __shared__ uint32_t idx[N];        // request index at each sorted position
  __shared__ uint32_t hp[N + 1];     // first sorted position of each group
  __shared__ uint32_t tiles[N + 1];  // tile prefix sums per group
  __shared__ uint64_t wsum[THREADS / 64];
  __shared__ uint32_t cnt[4];        // valid requests, error, tile slots used, items
  const uint32_t t = threadIdx.x, n = num_reqs, i0 = t * EPT;
  uint32_t *wsum32 = reinterpret_cast<uint32_t *>(wsum);
  uint32_t *heads = reinterpret_cast<uint32_t *>(swap + N);  // entry offsets of items, N + 1, after the sorts
  uint32_t half = 0;
  if (t >= 4u && t < 64u) work[t] = 0u;
  if (t < 4u) cnt[t] = 0u;
  __syncthreads();

  uint64_t key[EPT];
  bool valid[EPT], bad[EPT];
#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) {
    const uint32_t i = i0 + e;
    key[e] = ~0ull;
    valid[e] = bad[e] = false;
    if (i < n) {
      const xg_request q = reqs[i];
      valid[e] = q.stream < num_streams && q.dtype <= XG_NORMAL && q.flags == 0u;
      bad[e] = !valid[e];
      key[e] = ((valid[e] ? q.stream : 0xFFFFFFFFull) << 32) | i;
      costs[i] = cost_of(q.n, q.dtype);
    }
  }
  count_flags(valid, &cnt[0]);
  count_flags(bad, &cnt[1]);
  wg_sort<N, THREADS>(key, swap, half);
  __syncthreads();  // cnt and costs are written on every path by now

  const uint32_t valid_n = cnt[0];
  // Each thread's predecessor's last key: within the wavefront by a lane
  // shift, across wavefronts through LDS (idx is free until the keys go in).
  uint64_t before = __shfl_up(key[EPT - 1], 1u);
  if ((t & 63u) == 63u) wsum[t >> 6] = key[EPT - 1];
  __syncthreads();
  if ((t & 63u) == 0u && t) before = wsum[(t >> 6) - 1];
  uint32_t head[EPT], hx[EPT];
  uint64_t cx[EPT];
#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) {
    const uint32_t i = i0 + e;
    idx[i] = (uint32_t)key[e];
    head[e] = 0;
    cx[e] = 0;
    if (i < valid_n) {
      head[e] = i == 0 || (key[e] >> 32) != ((e ? key[e - 1] : before) >> 32);
      cx[e] = costs[(uint32_t)key[e]];
    }
    hx[e] = head[e];
  }
  __syncthreads();  // costs and wsum are rewritten below
  uint32_t num_groups;
  wg_exclusive<uint32_t, THREADS, EPT>(hx, wsum32, &num_groups);
  uint64_t cost_total;
  wg_exclusive<uint64_t, THREADS, EPT>(cx, wsum, &cost_total);
#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) {
    costs[i0 + e] = cx[e];
    if (i0 + e < n && head[e]) hp[hx[e]] = i0 + e;
  }
  if (t == 0) {
    costs[N] = cost_total;
    hp[num_groups] = valid_n;
  }
  __syncthreads();

  // tile_cap is the same on every thread.
  uint32_t used = 0;
  if (tile_cap) {
    uint32_t want[EPT];
#pragma unroll
    for (uint32_t e = 0; e < EPT; ++e) {
      const uint32_t g = i0 + e;
      want[e] = 0;
      if (g < num_groups && hp[g + 1] - hp[g] == 1u) {
        const xg_request q = reqs[idx[hp[g]]];
        const uint64_t parts = (words_of(q.n, q.dtype) + tile_words - 1) / tile_words;
        if (parts > 1 && parts <= kMaxSegments) want[e] = (uint32_t)parts;
      }
    }
    uint32_t tile_total;
    wg_exclusive<uint32_t, THREADS, EPT>(want, wsum32, &tile_total);
#pragma unroll
    for (uint32_t e = 0; e < EPT; ++e) {
      tiles[i0 + e] = want[e];
      if (want[e] && want[e] <= tile_cap) atomicMax(&cnt[2], want[e]);
    }
    if (t == 0) {
      tiles[N] = tile_total;
      if (tile_total && tile_total <= tile_cap) atomicMax(&cnt[2], tile_total);
    }
    __syncthreads();
    used = cnt[2];
  }
  auto is_split = [&](uint32_t g) { return tile_cap && group_split(tiles, g, used); };

  // Queue items: with tiles, by place in swap (the tiles' slots, then the
  // groups); without, group g on its own thread.
  uint32_t num_items;
  if (tile_cap) {
#pragma unroll
    for (uint32_t e = 0; e < EPT; ++e) swap[i0 + e] = ~0ull;
    __syncthreads();
#pragma unroll
    for (uint32_t e = 0; e < EPT; ++e) {
      const uint32_t g = i0 + e;
      if (g >= num_groups) continue;
      if (is_split(g)) {
        const xg_request q = reqs[idx[hp[g]]];
        const uint32_t parts = tiles[g + 1] - tiles[g];
        for (uint32_t k = 0; k < parts; ++k) {
          const uint64_t first = k * tile_words;
          const uint64_t nk = q.n - first < tile_words ? q.n - first : tile_words;
          swap[tiles[g] + k] = item_key(cost_of(nk, q.dtype), g, k);
        }
        atomicAdd(&cnt[3], parts);
      } else {
        swap[tile_cap + g] = item_key(costs[hp[g + 1]] - costs[hp[g]], g, 0);
        atomicAdd(&cnt[3], 1u);
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t e = 0; e < EPT; ++e) key[e] = swap[i0 + e];
    num_items = cnt[3];
    __syncthreads();  // the sort reuses swap
  } else {
#pragma unroll
    for (uint32_t e = 0; e < EPT; ++e) {
      const uint32_t g = i0 + e;
      key[e] = g < num_groups ? item_key(costs[hp[g + 1]] - costs[hp[g]], g, 0) : ~0ull;
    }
    num_items = num_groups;
  }
  wg_sort<N, THREADS>(key, swap, half);

  uint32_t ox[EPT];
#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) {
    const uint32_t q = i0 + e;
    ox[e] = 0;
    if (q < num_items) {
      const uint32_t g = (uint32_t)key[e] >> 8;
      ox[e] = is_split(g) ? 1u : hp[g + 1] - hp[g];
    }
  }
  uint32_t entries;
  wg_exclusive<uint32_t, THREADS, EPT>(ox, wsum32, &entries);
  const uint32_t items = n + tile_cap;
  __syncthreads();  // the sort's last reads of swap
#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) {
    heads[i0 + e] = ox[e];
    swap[i0 + e] = key[e];
    if (i0 + e <= items) offs_out[i0 + e] = ox[e];
  }
  if (t == THREADS - 1u) {
    heads[N] = entries;
    if (items == N) offs_out[N] = entries;
  }
  __syncthreads();

#pragma unroll
  for (uint32_t e = 0; e < EPT; ++e) {
    const uint32_t en = i0 + e;
    if (en >= entries) continue;
    uint32_t lo = 0, hi = num_items;  // heads[lo] <= en < heads[hi]
    while (hi - lo > 1u) {
      const uint32_t mid = (lo + hi) >> 1;
      if (heads[mid] <= en) lo = mid;
      else hi = mid;
    }
    const uint64_t it = swap[lo];
    const uint32_t g = (uint32_t)it >> 8, k = (uint32_t)it & 0xFFu;
    if (is_split(g)) {
      xg_request q = reqs[idx[hp[g]]];
      const uint64_t first = k * tile_words;
      const uint32_t parts = tiles[g + 1] - tiles[g], slot = tiles[g] + k;
      q.n = q.n - first < tile_words ? q.n - first : tile_words;
      q.out_offset += first;
      q.flags = kReqSegment | (k << 8) | (slot << 16) | (k + 1 == parts ? kReqLast : 0u);
      table[en] = q;
    } else {
      table[en] = reqs[idx[hp[g] + (en - heads[lo])]];
    }
  }
  if (t == 0) {
    work[0] = 0u;
    work[1] = cnt[1] ? 1u : 0u;
    work[2] = num_items;
    work[3] = entries;
  }
}

uint32_t pow2_at_least(uint32_t v) {
  uint32_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace

PlanLayout plan_layout(uint32_t max_reqs, uint32_t max_tiles, uint32_t state_bytes, uint32_t jump_bytes) {
  PlanLayout l;
  l.key_cap = pow2_at_least(max_reqs > kLeastKeys ? max_reqs : kLeastKeys);
  const uint32_t items = max_reqs + max_tiles;
  l.item_cap = pow2_at_least(items > kLeastKeys ? items : kLeastKeys);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = align256(o + bytes);
    return at;
  };
  l.work = take(256);
  l.meta = take(256);
  l.keys = take((size_t)l.key_cap * 8);
  l.heads = take(((size_t)max_reqs + 1) * 4);
  l.costs = take(((size_t)max_reqs + 1) * 8);
  l.hp = take(((size_t)max_reqs + 1) * 4);
  l.tiles = take(((size_t)max_reqs + 1) * 4);
  l.items = take((size_t)l.item_cap * 8);
  l.offs = take(((size_t)items + 1) * 4);
  l.table = take((size_t)items * sizeof(xg_request));
  l.sums = take(1024 * 8);
  l.stage = take((size_t)max_tiles * state_bytes);
  l.jump = take(max_tiles ? (size_t)(kMaxSegments - 1) * jump_bytes : 0);
  l.total = o;
  return l;
}

PlanPtrs plan_ptrs(void *base, const PlanLayout &l) {
  char *b = static_cast<char *>(base);
  PlanPtrs p;
  p.work = reinterpret_cast<uint32_t *>(b + l.work);
  p.meta = reinterpret_cast<uint32_t *>(b + l.meta);
  p.keys = reinterpret_cast<uint64_t *>(b + l.keys);
  p.heads = reinterpret_cast<uint32_t *>(b + l.heads);
  p.costs = reinterpret_cast<uint64_t *>(b + l.costs);
  p.hp = reinterpret_cast<uint32_t *>(b + l.hp);
  p.tiles = reinterpret_cast<uint32_t *>(b + l.tiles);
  p.items = reinterpret_cast<uint64_t *>(b + l.items);
  p.offs = reinterpret_cast<uint32_t *>(b + l.offs);
  p.table = reinterpret_cast<xg_request *>(b + l.table);
  p.sums = reinterpret_cast<uint64_t *>(b + l.sums);
  p.stage = reinterpret_cast<uint32_t *>(b + l.stage);
  p.jump = reinterpret_cast<uint64_t *>(b + l.jump);
  return p;
}

hipError_t launch_plan(const PlanPtrs &p, const PlanLayout &l, const xg_request *reqs, uint32_t num_reqs,
                       uint64_t num_streams, uint64_t tile_words, uint32_t max_tiles, hipStream_t stream) {
  const uint32_t tile_cap = tile_words ? max_tiles : 0u;
  const uint64_t elems = (uint64_t)num_reqs + tile_cap;
  if (elems <= kSmallPlanMax) {
    if (elems + 1 > (uint64_t)(l.table - l.offs) / 4) return hipErrorInvalidValue;
    auto run = [&](auto kernel, uint32_t threads) {
      return launch(kernel, dim3(1), dim3(threads), 0, stream, reqs, num_reqs, num_streams, tile_words, tile_cap,
                    p.work, p.offs, p.table);
    };
    if (elems <= 256) return run(k_plan_small<256, 256>, 256);
    if (elems <= 512) return run(k_plan_small<512, 512>, 512);
    if (elems <= 1024) return run(k_plan_small<1024, 1024>, 1024);
    if (elems <= 2048) return run(k_plan_small<2048, 1024>, 1024);
    return run(k_plan_small<4096, 1024>, 1024);
  }
  const uint32_t key_n = pow2_at_least(num_reqs > kLeastKeys ? num_reqs : kLeastKeys);
  const uint32_t items = num_reqs + tile_cap;
  const uint32_t item_n = pow2_at_least(items > kLeastKeys ? items : kLeastKeys);
  // The sorts' second buffer is the table, which the last step writes; the
  // head sums lie in offs, which the items' counts fill later.
  const uint32_t sorted = key_n > item_n ? key_n : item_n;
  if (key_n > l.key_cap || item_n > l.item_cap || items > kPlanMaxElems ||
      (uint64_t)sorted * 8 > l.sums - l.table || l.table - l.offs < 1024 * 4)
    return hipErrorInvalidValue;
  const dim3 b256(256);
  auto grid = [](uint32_t n) { return dim3(n ? (n + 255) / 256 : 1u); };
  auto scan_grid = [](uint32_t n) { return dim3(n ? (n + kScanBlock - 1) / kScanBlock : 1u); };
  uint64_t *tmp = reinterpret_cast<uint64_t *>(p.table);
  uint32_t *u32sums = reinterpret_cast<uint32_t *>(p.sums);
  hipError_t e = sort_keys(p.keys, tmp, key_n, reqs, num_reqs, num_streams, p.work, p.meta, stream);
  if (e == hipSuccess)
    e = launch(k_plan_heads, scan_grid(num_reqs), b256, 0, stream, reqs, num_reqs, p.keys, p.meta, p.work, p.heads,
               p.costs, p.offs, p.sums);
  if (e == hipSuccess)
    e = launch(k_plan_groups, scan_grid(num_reqs), b256, 0, stream, num_reqs, p.heads, p.costs, p.offs, p.sums,
               p.meta, p.hp, tile_cap ? nullptr : p.tiles, p.items, item_n);
  if (tile_cap) {
    if (e == hipSuccess)
      e = launch(k_plan_want, scan_grid(num_reqs), b256, 0, stream, reqs, num_reqs, p.keys, p.heads, p.hp,
                 tile_words, p.tiles, u32sums);
    if (e == hipSuccess)
      e = launch(k_plan_budget, scan_grid(num_reqs), b256, 0, stream, num_reqs, p.tiles, u32sums, tile_cap, p.meta);
  }
  if (e == hipSuccess)
    e = launch(k_plan_items, grid(num_reqs), b256, 0, stream, reqs, num_reqs, p.keys, p.heads, p.costs, p.hp,
               p.tiles, tile_words, tile_cap, p.meta, p.items);
  if (e == hipSuccess) e = sort_keys(p.items, tmp, item_n, nullptr, 0, 0, p.work, p.meta, stream);
  if (e == hipSuccess)
    e = launch(k_plan_counts, scan_grid(items), b256, 0, stream, items, p.items, p.hp, p.tiles, p.meta, p.offs,
               u32sums);
  if (e == hipSuccess) e = launch(k_scan, scan_grid(items), b256, 0, stream, p.offs, items, u32sums);
  if (e == hipSuccess)
    e = launch(k_plan_emit, grid(items), b256, 0, stream, reqs, p.keys, p.hp, p.tiles, tile_words, p.items, items,
               p.offs, p.meta, p.table, p.work);
  return e;
}

}  // namespace xg
