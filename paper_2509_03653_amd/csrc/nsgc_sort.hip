// Device-wide stable LSD radix sort of 64-bit keys, and an exclusive scan.
// Used where a window or a whole batch is too large for LDS hashing to
// aggregate in one partitioning level (large windows that hash partitioning
// gives up on, and the address anonymization).
//
// One pass sorts by an 8-bit digit (the last may be narrower) over up to 512
// contiguous ranges of the keys, two workgroups per compute unit:
//   1. the digit histogram of every range, digit-major ([digit][range]);
//   2. an exclusive scan of every digit's row, and the digits' totals;
//   3. a scatter in which each workgroup carries its range's 256 positions
//      from tile to tile.  Every wavefront ranks its consecutive keys of the
//      tile (64 a round, in order) among equal digits with ballots, so the
//      order within a tile is kept too; the tile is put in digit order in LDS
//      and leaves in runs, 32 keys on average.
// Passes ping-pong between the key buffer and a second buffer of equal size.
// The number of keys may be known on the device only.
//
// Bound by the ballots and LDS of the ranking.  A pass over 7 * 10^6 keys takes
// 55 us (hist 15, rows 5, scatter 35: 3.2 TB/s); with a histogram per tile of
// 4096 keys, three launches to scan those and keys written straight to their
// places a pass over 1.7 * 10^7 took 175.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

#include "nsgc_device.hpp"
#include "nsgc_ranges.hpp"
#include "nsgc_sort.hpp"

namespace nsgc {

namespace {

constexpr uint32_t RS_THREADS = 512;
constexpr uint32_t RS_PER = 8;                       // elements per thread of a scan block
constexpr uint32_t RS_WAVES = RS_THREADS / 64;
constexpr uint32_t RS_RANGES = 512;                  // most ranges of a pass
static_assert(RS_RANGES == RS_THREADS, "a thread per range scans a digit's row");
constexpr uint32_t SCAN_TILE = RS_THREADS * RS_PER;  // elements per scan block

__device__ __forceinline__ uint32_t digit_of(u64 k, uint32_t shift, uint32_t mask) {
  return uint32_t(k >> shift) & mask;
}

// Keys, and the range of this workgroup: whole tiles, the same for every
// kernel of a pass.
__device__ __forceinline__ ListRange my_range(u64 n, const uint32_t* ndev, uint32_t chunk) {
  return list_range(ndev ? *ndev : n, chunk, gridDim.x, blockIdx.x);
}

__global__ __launch_bounds__(RS_THREADS) void k_rs_hist(const u64* __restrict__ keys, u64 n,
                                                        const uint32_t* ndev, uint32_t chunk, uint32_t shift,
                                                        uint32_t bits, uint32_t* __restrict__ counts) {
  __shared__ uint32_t hist[RS_WAVES][256];
  const ListRange R = my_range(n, ndev, chunk);
  const uint32_t mask = (1u << bits) - 1u, tid = threadIdx.x;
  for (uint32_t i = tid; i < RS_WAVES * 256; i += RS_THREADS) (&hist[0][0])[i] = 0;
  __syncthreads();
  uint32_t* const h = hist[tid >> 6];
  for (u64 base = R.beg; base < R.end; base += RS_THREADS * 8) {
    u64 key[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const u64 i = base + k * RS_THREADS + tid;
      key[k] = i < R.end ? keys[i] : 0ull;
    }
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)
      if (base + k * RS_THREADS + tid < R.end) lds_add(&h[digit_of(key[k], shift, mask)], 1);
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t s = 0;
#pragma unroll
    for (uint32_t w = 0; w < RS_WAVES; ++w) s += hist[w][tid];
    counts[tid * gridDim.x + blockIdx.x] = s;
  }
}

// A digit's row of counts (at most one per thread) to its exclusive prefix, and
// its total.
__global__ __launch_bounds__(RS_THREADS) void k_rs_rows(uint32_t* __restrict__ counts, uint32_t ranges,
                                                        uint32_t* __restrict__ totals) {
  __shared__ uint32_t red[RS_WAVES];
  const uint32_t tid = threadIdx.x, w = tid >> 6;
  uint32_t* const row = counts + blockIdx.x * ranges;
  const uint32_t x = tid < ranges ? row[tid] : 0u;
  const uint32_t incl = wave_inclusive_scan(x);
  if (lane_id() == 63) red[w] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (uint32_t k = 0; k < RS_WAVES; ++k) {
    if (k < w) before += red[k];
    all += red[k];
  }
  if (tid < ranges) row[tid] = before + incl - x;
  if (tid == 0) totals[blockIdx.x] = all;
}

// Scan, first level: the sum of every block of SCAN_TILE elements.
__global__ __launch_bounds__(RS_THREADS) void k_scan_reduce(const uint32_t* __restrict__ a, u64 n,
                                                            uint32_t* __restrict__ bsum) {
  __shared__ uint32_t red[RS_WAVES];
  const u64 base = u64(blockIdx.x) * SCAN_TILE;
  uint32_t s = 0;
#pragma unroll
  for (uint32_t k = 0; k < RS_PER; ++k) {
    const u64 i = base + u64(k) * RS_THREADS + threadIdx.x;
    if (i < n) s += a[i];
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) bsum[blockIdx.x] = s;
}

// Scan, second level: exclusive scan of the block sums in one workgroup.
__global__ __launch_bounds__(RS_THREADS) void k_scan_top(uint32_t* __restrict__ bsum, uint32_t nb) {
  __shared__ uint32_t red[RS_WAVES];
  __shared__ uint32_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (uint32_t c0 = 0; c0 < nb; c0 += RS_THREADS) {
    const uint32_t i = c0 + threadIdx.x;
    const uint32_t v = i < nb ? bsum[i] : 0u;
    const uint32_t incl = wave_inclusive_scan(v);
    const uint32_t w = threadIdx.x >> 6;
    if (lane_id() == 63) red[w] = incl;
    __syncthreads();
    uint32_t before = carry, total = 0;
    for (uint32_t k = 0; k < RS_WAVES; ++k) {
      if (k < w) before += red[k];
      total += red[k];
    }
    if (i < nb) bsum[i] = before + incl - v;
    __syncthreads();
    if (threadIdx.x == 0) carry += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[nb] = carry;   // the grand total, after the block prefixes
}

// Scan, third level: each block's elements in place, offset by its block's
// exclusive prefix.  Thread t takes RS_PER consecutive elements.
__global__ __launch_bounds__(RS_THREADS) void k_scan_down(uint32_t* __restrict__ a, u64 n,
                                                          const uint32_t* __restrict__ bsum) {
  __shared__ uint32_t red[RS_WAVES];
  const u64 base = u64(blockIdx.x) * SCAN_TILE + u64(threadIdx.x) * RS_PER;
  uint32_t v[RS_PER];
  uint32_t s = 0;
#pragma unroll
  for (uint32_t k = 0; k < RS_PER; ++k) {
    v[k] = base + k < n ? a[base + k] : 0u;
    s += v[k];
  }
  const uint32_t incl = wave_inclusive_scan(s);
  const uint32_t w = threadIdx.x >> 6;
  if (lane_id() == 63) red[w] = incl;
  __syncthreads();
  uint32_t run = bsum[blockIdx.x] + incl - s;
  for (uint32_t k = 0; k < w; ++k) run += red[k];
#pragma unroll
  for (uint32_t k = 0; k < RS_PER; ++k) {
    if (base + k < n) a[base + k] = run;
    run += v[k];
  }
}

// ROUNDS: keys per thread of a tile.
template <uint32_t ROUNDS>
__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(const u64* __restrict__ in, u64* __restrict__ out,
                                                           u64 n, const uint32_t* ndev, uint32_t shift,
                                                           uint32_t bits, const uint32_t* __restrict__ counts,
                                                           const uint32_t* __restrict__ totals) {
  constexpr uint32_t CHUNK = RS_THREADS * ROUNDS;
  __shared__ u64 stage[CHUNK];
  __shared__ uint32_t cnt[RS_WAVES][256];
  __shared__ uint32_t to[256];      // output position of the digit's next key, less its place in the tile
  __shared__ uint32_t red[4];
  const ListRange R = my_range(n, ndev, CHUNK);
  const uint32_t mask = (1u << bits) - 1u, tid = threadIdx.x, w = tid >> 6, lane = lane_id();
  uint32_t pos = 0;                 // of digit `tid`: the range's next position
  if (tid < 256) {
    const uint32_t x = totals[tid], incl = wave_inclusive_scan(x);
    if (lane == 63) red[w] = incl;
    pos = incl - x + counts[tid * gridDim.x + blockIdx.x];
  }
  __syncthreads();
  if (tid < 256)
    for (uint32_t k = 0; k < w; ++k) pos += red[k];
  for (u64 base = R.beg; base < R.end; base += CHUNK) {
    const uint32_t len = uint32_t(min(u64(CHUNK), R.end - base));
    __syncthreads();
    for (uint32_t i = lane; i < 256; i += 64) cnt[w][i] = 0;
    u64 key[ROUNDS];
    uint32_t rk[ROUNDS];
    const uint32_t w0 = w * (ROUNDS * 64) + lane;
#pragma unroll
    for (uint32_t r = 0; r < ROUNDS; ++r) key[r] = w0 + r * 64 < len ? in[base + w0 + r * 64] : 0ull;
#pragma unroll
    for (uint32_t r = 0; r < ROUNDS; ++r) {
      const bool ok = w0 + r * 64 < len;
      const uint32_t d = digit_of(key[r], shift, mask);
      // lanes with the same digit: intersect the ballots of its bits
      u64 m = __ballot(ok);
#pragma unroll
      for (uint32_t b = 0; b < 8; ++b) {   // (bits above the digit's are zero in every lane)
        const u64 mb = __ballot((d >> b) & 1u);
        m &= ((d >> b) & 1u) ? mb : ~mb;
      }
      const uint32_t leader = ok ? uint32_t(__ffsll(static_cast<unsigned long long>(m)) - 1) : 0u;
      uint32_t old = 0;
      if (ok && lane == leader) old = lds_add(&cnt[w][d], uint32_t(__popcll(m)));
      rk[r] = lane_take(old, leader) + rank_below(m);
    }
    __syncthreads();
    // a digit's counts by wavefront to places in the tile
    uint32_t mine = 0, incl = 0;
    if (tid < 256) {
#pragma unroll
      for (uint32_t k = 0; k < RS_WAVES; ++k) {
        const uint32_t c = cnt[k][tid];
        cnt[k][tid] = mine;
        mine += c;
      }
      incl = wave_inclusive_scan(mine);
      if (lane == 63) red[w] = incl;
    }
    __syncthreads();
    if (tid < 256) {
      uint32_t first = incl - mine;
      for (uint32_t k = 0; k < w; ++k) first += red[k];
#pragma unroll
      for (uint32_t k = 0; k < RS_WAVES; ++k) cnt[k][tid] += first;
      to[tid] = pos - first;
      pos += mine;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < ROUNDS; ++r)
      if (w0 + r * 64 < len) stage[cnt[w][digit_of(key[r], shift, mask)] + rk[r]] = key[r];
    __syncthreads();
    for (uint32_t i = tid; i < len; i += RS_THREADS) {
      const u64 k = stage[i];
      out[u64(to[digit_of(k, shift, mask)] + i)] = k;
    }
  }
}

}  // namespace

size_t scan_scratch_words(u64 n) { return size_t((n + SCAN_TILE - 1) / SCAN_TILE) + 64; }

size_t radix_sort_scratch_words() { return 256 * RS_RANGES + 256; }

uint32_t* scan_total(uint32_t* bsum, u64 n) { return bsum + (n + SCAN_TILE - 1) / SCAN_TILE; }

hipError_t exclusive_scan_u32(uint32_t* a, u64 n, uint32_t* bsum, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const u64 nb = (n + SCAN_TILE - 1) / SCAN_TILE;
  if (nb > 0xFFFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_scan_reduce, dim3(uint32_t(nb)), dim3(RS_THREADS), 0, s, a, n, bsum);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(RS_THREADS), 0, s, bsum, uint32_t(nb));
  hipLaunchKernelGGL(k_scan_down, dim3(uint32_t(nb)), dim3(RS_THREADS), 0, s, a, n, bsum);
  return hipGetLastError();
}

hipError_t radix_sort_u64(u64* keys, u64* tmp, u64 n, const uint32_t* ndev, uint32_t lo, uint32_t hi,
                          uint32_t* scratch, hipStream_t s, u64** sorted) {
  *sorted = keys;
  if (n <= 1 || hi <= lo) return hipSuccess;
  // Tiles of four keys per thread while they fit the ranges: each of a pass'
  // few tiles is a serial chain (8 * 10^4 keys: 10 us a scatter with sixteen, 5
  // with four).
  const bool few = n <= u64(RS_RANGES) * RS_THREADS * 4;
  const uint32_t chunk = RS_THREADS * (few ? 4 : 16);
  const uint32_t ranges = uint32_t(std::min<u64>((n + chunk - 1) / chunk, RS_RANGES));
  uint32_t* counts = scratch;
  uint32_t* totals = scratch + 256 * RS_RANGES;
  u64* a = keys;
  u64* b = tmp;
  for (uint32_t shift = lo; shift < hi; shift += 8) {
    const uint32_t bits = std::min(8u, hi - shift);
    hipLaunchKernelGGL(k_rs_hist, dim3(ranges), dim3(RS_THREADS), 0, s, a, n, ndev, chunk, shift, bits,
                       counts);
    hipLaunchKernelGGL(k_rs_rows, dim3(256), dim3(RS_THREADS), 0, s, counts, ranges, totals);
    if (few)
      hipLaunchKernelGGL((k_rs_scatter<4>), dim3(ranges), dim3(RS_THREADS), 0, s, a, b, n, ndev, shift, bits,
                         counts, totals);
    else
      hipLaunchKernelGGL((k_rs_scatter<16>), dim3(ranges), dim3(RS_THREADS), 0, s, a, b, n, ndev, shift, bits,
                         counts, totals);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    std::swap(a, b);
  }
  *sorted = a;
  return hipSuccess;
}

}  // namespace nsgc
