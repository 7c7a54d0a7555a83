// Address anonymization on the device (Section IV, "IP Address
// Anonymization"): every address of the source and destination columns is
// replaced by a distinct integer in [0, N), N the number of unique addresses,
// through a seeded permutation of 0..N-1.
//
// The unique addresses are listed in ascending order and the i-th one maps to
// pi(i), where pi is a keyed pseudo-random permutation of [0, N): a
// four-round Feistel network on the smallest even bit count b with 2^b >=
// max(N, 4), round function F_r(R) = mix(seed ^ (r + 1) * 0x9E3779B97F4A7C15
// ^ R) on the low b/2 bits (mix = the SplitMix64 output function), restricted
// to [0, N) by cycle walking (Black and Rogaway, 2002).  A Feistel network is
// a bijection for any round function, so pi is one too.
//
// On the device, the paper's unique / shuffle / gather sorts each tile's
// distinct addresses only:
//   1. k_an_tiles finds the distinct addresses of every tile of 2^14 entries of
//      a column in an LDS table, lists them as (address << 32 | place in the
//      list) and writes every entry's index among its tile's;
//   2. a stable radix sort by the address half brings equal addresses
//      together, in ascending order;
//   3. k_an_starts counts the runs of equal addresses in each of 512 ranges,
//      and k_an_values numbers them (the rank i) and writes pi(i) to the
//      element's place in the list;
//   4. k_an_apply replaces every entry's index by its tile's value.
//
// Sorting every entry with its position moved 16 bytes per entry in each of
// four passes and scattered the results over the columns, 1046 us for two
// columns of 2^23; tiles have 0.3 to 0.5 distinct addresses per entry of
// heavy-tailed traffic, and it takes 427 (tiles 70, sort 220, values 122, whose
// 4-byte writes to random places bound it, apply 21).  Two columns of 3371: 90
// -> 64, launches.
#include <hip/hip_runtime.h>

#include "nsgc_anon.hpp"
#include "nsgc_device.hpp"
#include "nsgc_ranges.hpp"
#include "nsgc_sort.hpp"

namespace nsgc {

namespace {

constexpr uint32_t NT = 1024;                // threads of the tile kernels
constexpr uint32_t PER = 16;                 // entries per thread
constexpr uint32_t TILE = NT * PER;          // entries per tile; their indexes take 16 bits
constexpr uint32_t SLOTS = 2 * TILE;
constexpr uint32_t VT = 512;                 // threads of the range kernels
constexpr uint32_t RANGES = 512;             // most ranges
static_assert(RANGES == VT, "a thread per range adds up their counts");

struct Tile {
  uint32_t first, count;   // its distinct addresses' place in the list
};

// The column and the entries of tile t: the first half of the tiles are the
// source column's.
struct Part {
  uint32_t dst, beg, len;
  __device__ Part(uint32_t t, uint32_t tiles, uint32_t n) {
    dst = t >= tiles;
    beg = (t - (dst ? tiles : 0u)) * TILE;
    len = min(TILE, n - beg);
  }
};

// The table fills at most half.  Its slots hold addresses, then their indexes
// within the tile; address 0xFFFFFFFF, the free mark, is kept beside it.
__global__ __launch_bounds__(NT) void k_an_tiles(const uint32_t* __restrict__ src, const uint32_t* __restrict__ dst,
                                                 uint32_t n, uint32_t tiles, u64* __restrict__ list,
                                                 uint32_t* total, Tile* __restrict__ meta,
                                                 uint16_t* __restrict__ index) {
  extern __shared__ __align__(16) uint32_t table[];   // [SLOTS]
  __shared__ uint32_t misc[3];   // distinct addresses, 1 + index of 0xFFFFFFFF, place in the list
  const uint32_t tid = threadIdx.x;
  const Part P(blockIdx.x, tiles, n);
  const NSGC_GLOBAL uint32_t* in = gptr(P.dst ? dst : src) + P.beg;
  uint32_t a[PER], at[PER];
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) a[k] = in[min(k * NT + tid, P.len - 1)];
  const v4u32 e4 = {EMPTY32, EMPTY32, EMPTY32, EMPTY32};
#pragma unroll
  for (uint32_t i = 0; i < SLOTS / 4 / NT; ++i) reinterpret_cast<v4u32*>(table)[i * NT + tid] = e4;
  if (tid < 3) misc[tid] = 0;
  lds_barrier();
  uint32_t own = 0;   // entries that inserted their address
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) {
    at[k] = SLOTS;    // 0xFFFFFFFF
    if (k * NT + tid < P.len && a[k] != EMPTY32) {
      uint32_t s = row_hash(a[k]) & (SLOTS - 1);
      for (;;) {      // ends: the table has twice as many slots as the tile has entries
        const uint32_t old = lds_cas32(&table[s], EMPTY32, a[k]);
        if (old == EMPTY32) own |= 1u << k;
        if (old == EMPTY32 || old == a[k]) break;
        s = (s + 1) & (SLOTS - 1);
      }
      at[k] = s;
    } else if (k * NT + tid < P.len) {
      misc[1] = 1;
    }
  }
  lds_barrier();
  // indexes: each wavefront's inserted addresses in turn
  const uint32_t mine = __popc(own), incl = wave_inclusive_scan(mine);
  uint32_t base = 0;
  if (lane_id() == 63) base = lds_add(&misc[0], incl);
  base = readlane(base, 63) + incl - mine;
  uint32_t next = base;
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k)
    if (own >> k & 1u) table[at[k]] = next++;
  lds_barrier();
  if (tid == 0) {
    uint32_t count = misc[0];
    if (misc[1]) misc[1] = ++count;
    const uint32_t first = __hip_atomic_fetch_add(total, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    meta[blockIdx.x] = {first, count};
    misc[2] = first;
    if (misc[1]) list[first + count - 1] = (u64(EMPTY32) << 32) | (first + count - 1);
  }
  NSGC_GLOBAL uint16_t* out = gptr(index) + (P.dst ? u64(n) : 0ull) + P.beg;
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k)
    if (k * NT + tid < P.len && at[k] != SLOTS) out[k * NT + tid] = uint16_t(table[at[k]]);
  lds_barrier();
  const uint32_t first = misc[2];
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) {
    if (own >> k & 1u) {
      list[first + base] = (u64(a[k]) << 32) | (first + base);
      ++base;
    }
    if (k * NT + tid < P.len && at[k] == SLOTS) out[k * NT + tid] = uint16_t(misc[1] - 1u);
  }
}

// This workgroup's part of the sorted list (up to 2^32 - 2 elements), in whole
// steps of 64 elements per wavefront.
__device__ __forceinline__ ListRange my_range(uint32_t m) { return list_range(m, VT, gridDim.x, blockIdx.x); }

// Whether element i of the sorted list starts a run of equal addresses.
__device__ __forceinline__ bool run_start(const u64* s, uint32_t i) {
  return i == 0 || (s[i] >> 32) != (s[i - 1] >> 32);
}

__global__ __launch_bounds__(VT) void k_an_starts(const u64* __restrict__ s, const uint32_t* __restrict__ total,
                                                  uint32_t* __restrict__ starts) {
  __shared__ uint32_t red[VT / 64];
  const ListRange R = my_range(*total);
  uint32_t c = 0;
#pragma unroll 4
  for (u64 i = R.beg + threadIdx.x; i < R.end; i += VT) c += run_start(s, uint32_t(i));
  c = block_sum(c, red);
  if (threadIdx.x == 0) starts[blockIdx.x] = c;
}

__device__ __forceinline__ u64 sm_out(u64 z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// The Feistel permutation of [0, 2^(2h)) for `seed`.
__device__ __forceinline__ u64 feistel_e(u64 x, uint32_t h, u64 seed) {
  const u64 mask = (u64(1) << h) - 1;
  u64 lo = x & mask, hi = x >> h;
#pragma unroll
  for (u64 r = 1; r <= 4; ++r) {
    const u64 t = hi ^ (sm_out(seed ^ (r * 0x9E3779B97F4A7C15ull) ^ lo) & mask);
    hi = lo;
    lo = t;
  }
  return (hi << h) | lo;
}

// Each element: its address's rank among the unique ones (run starts up to it,
// less one), through the permutation, to its place in the list.
__global__ __launch_bounds__(VT) void k_an_values(const u64* __restrict__ s, const uint32_t* __restrict__ total,
                                                  const uint32_t* __restrict__ starts, u64 seed,
                                                  uint32_t* __restrict__ values,
                                                  unsigned long long* __restrict__ num) {
  constexpr uint32_t VU = 8;   // elements of a thread in flight
  __shared__ uint32_t red[2][VT / 64];
  __shared__ uint32_t step[VU][VT / 64];
  const uint32_t tid = threadIdx.x, w = tid >> 6;
  const uint32_t c = tid < gridDim.x ? starts[tid] : 0u;
  const uint32_t all = wave_sum(c), below = wave_sum(tid < blockIdx.x ? c : 0u);
  if (lane_id() == 0) {
    red[0][w] = all;
    red[1][w] = below;
  }
  __syncthreads();
  uint32_t before = 0;
  u64 N = 0;
#pragma unroll
  for (uint32_t k = 0; k < VT / 64; ++k) {
    N += red[0][k];
    before += red[1][k];
  }
  uint32_t h = 1;                       // b = 2h: the smallest even b with 2^b >= max(N, 4)
  while ((u64(1) << (2 * h)) < N) ++h;
  const ListRange R = my_range(*total);
  for (u64 i0 = R.beg; i0 < R.end; i0 += VU * VT) {
    u64 x[VU], m[VU];
    bool in[VU], start[VU];
#pragma unroll
    for (uint32_t u = 0; u < VU; ++u) {
      const u64 i = i0 + u * VT + tid;
      in[u] = i < R.end;
      x[u] = s[in[u] ? i : R.beg];
      start[u] = in[u] && (i == 0 || (s[i - 1] >> 32) != (x[u] >> 32));
    }
#pragma unroll
    for (uint32_t u = 0; u < VU; ++u) {
      m[u] = __ballot(start[u]);
      if (lane_id() == 0) step[u][w] = __popcll(m[u]);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < VU; ++u) {
      uint32_t at = before;
#pragma unroll
      for (uint32_t k = 0; k < VT / 64; ++k) {
        const uint32_t y = step[u][k];
        if (k < w) at += y;
        before += y;
      }
      if (in[u]) {
        const u64 rank = u64(at + rank_below(m[u]) + (start[u] ? 1u : 0u)) - 1u;
        u64 y = rank;
        if (N > 1) {
          y = feistel_e(rank, h, seed);
          while (y >= N) y = feistel_e(y, h, seed);
        }
        values[uint32_t(x[u])] = uint32_t(y);
      }
    }
    __syncthreads();
  }
  if (blockIdx.x == 0 && tid == 0) *num = N;
}

__global__ __launch_bounds__(NT) void k_an_apply(uint32_t n, uint32_t tiles, const Tile* __restrict__ meta,
                                                 const uint16_t* __restrict__ index,
                                                 const uint32_t* __restrict__ values, uint32_t* __restrict__ asrc,
                                                 uint32_t* __restrict__ adst) {
  __shared__ uint32_t v[TILE];
  const uint32_t tid = threadIdx.x;
  const Part P(blockIdx.x, tiles, n);
  const NSGC_GLOBAL uint16_t* in = gptr(index) + (P.dst ? u64(n) : 0ull) + P.beg;
  uint32_t x[PER];
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k) x[k] = in[min(k * NT + tid, P.len - 1)];
  const Tile M = meta[blockIdx.x];
  for (uint32_t i = tid; i < M.count; i += NT) v[i] = gptr(values)[M.first + i];
  __syncthreads();
  NSGC_GLOBAL uint32_t* out = gptr(P.dst ? adst : asrc) + P.beg;
#pragma unroll
  for (uint32_t k = 0; k < PER; ++k)
    if (k * NT + tid < P.len) out[k * NT + tid] = v[x[k]];
}

__global__ void k_an_zero(unsigned long long* num, uint32_t* total) {
  if (threadIdx.x == 0) {
    *num = 0;
    if (total) *total = 0;
  }
}

}  // namespace

size_t anonymize_bytes(u64 n) {
  const u64 m = 2 * n, tiles = 2 * ((n + TILE - 1) / TILE);
  const size_t words = size_t(m / 2) + 2 * size_t(tiles) + RANGES + radix_sort_scratch_words() + 64;
  return size_t(m) * 16 + words * 4 + 1024;
}

hipError_t anonymize_allow_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_an_tiles),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(SLOTS * 4));
}

hipError_t anonymize(const uint32_t* src, const uint32_t* dst, u64 n, u64 seed, uint32_t* asrc,
                     uint32_t* adst, unsigned long long* num, void* ws, hipStream_t s) {
  if (n == 0) {
    hipLaunchKernelGGL(k_an_zero, dim3(1), dim3(64), 0, s, num, static_cast<uint32_t*>(nullptr));
    return hipGetLastError();
  }
  const u64 m = 2 * n;
  u64* V = static_cast<u64*>(ws);
  u64* T = V + m;
  uint32_t* total = reinterpret_cast<uint32_t*>(T + m);
  uint32_t* starts = total + 16;
  uint32_t* scratch = starts + RANGES;
  const uint32_t tiles = uint32_t((n + TILE - 1) / TILE);
  Tile* meta = reinterpret_cast<Tile*>(scratch + radix_sort_scratch_words());
  uint16_t* index = reinterpret_cast<uint16_t*>(meta + 2 * tiles);
  hipError_t e;
  hipLaunchKernelGGL(k_an_zero, dim3(1), dim3(64), 0, s, num, total);
  hipLaunchKernelGGL(k_an_tiles, dim3(2 * tiles), dim3(NT), SLOTS * 4, s, src, dst, uint32_t(n), tiles, V, total,
                     meta, index);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  u64* S = nullptr;
  if ((e = radix_sort_u64(V, T, m, total, 32, 64, scratch, s, &S)) != hipSuccess) return e;
  uint32_t* values = reinterpret_cast<uint32_t*>(S == V ? T : V);   // the other buffer is free
  const uint32_t ranges = uint32_t(std::min<u64>((m + VT - 1) / VT, RANGES));
  hipLaunchKernelGGL(k_an_starts, dim3(ranges), dim3(VT), 0, s, S, total, starts);
  hipLaunchKernelGGL(k_an_values, dim3(ranges), dim3(VT), 0, s, S, total, starts, seed, values, num);
  hipLaunchKernelGGL(k_an_apply, dim3(2 * tiles), dim3(NT), 0, s, uint32_t(n), tiles, meta, index, values, asrc,
                     adst);
  return hipGetLastError();
}

}  // namespace nsgc
