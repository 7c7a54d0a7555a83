// Grid windows: statistics of the partitioned windows of more than 2^13
// packets (layout and the treatment of dominant addresses: nsgc_plan.h).
//
// k_grid_heavy samples each window for dominant addresses, k_grid_partition
// orders the window's hashed link keys by cell, k_grid_links counts each cell's
// links and emits their row and column entries, and k_grid_rowcol adds those up
// per source and per destination; k_grid_rounds and k_grid_sweeps finish the
// cells and buckets that are too large for one pass.  k_finish combines the
// totals.
//
// Against one link bucket per hash range (nsgc_kernels.hip): a cell's links
// fall into the one to a few row and column buckets of its two strips instead
// of every row and column bucket of the window, so its entries leave in long
// runs, need next to no per-bucket counting, and phase C reads a few long
// segments instead of one short one per link bucket.  Heavy-tailed traffic
// has up to half of its packets between dominant addresses; those are counted
// in LDS during the partition.
//
// Measured against that path, whole calls: 64 windows of 2^17 packets 237 ->
// 202 us; one of 40013 packets 58 -> 39 us; nine of 2^12 .. 2^22 packets 434 ->
// 165 us; 512 of 2^10 .. 2^23 packets 11.5 -> 7.1 ms; 128 of 2^23 14.2 -> 9.5
// ms; one of 2^20 with all addresses distinct 680 -> 128 us, among 4096 152 ->
// 92.  Slower is a window of 2^20 to 2^22 packets among 65 to a thousand
// addresses, whose few links one link bucket per range counts in fewer launches
// (one of 2^20 among 300 56 -> 85 us, eight 150 -> 176; among 2000 150 -> 94).
// Windows of up to 2^13 packets have one workgroup each.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "nsgc_device.hpp"
#include "nsgc_grid.hpp"
#include "nsgc_grid_device.hpp"
#include "nsgc_phases.hpp"
#include "nsgc_plan.h"

namespace nsgc {

namespace {

constexpr uint32_t HVM = NSGC_GRID_HEAVY;   // most dominant addresses per view

// Find-or-insert of U keys per lane in an open-addressing LDS table (probed like
// probe_on): the home slots of all U are tried together, then the keys still
// without a slot probe on in step, a key's turn being skipped when no lane
// needs it.  slot[u] comes in as the home slot and goes out as the key's slot;
// fr[u]: this call inserted the key.  Call with the whole wavefront active;
// returns whether a key of this lane found no slot.
template <int U, class K>
__device__ __forceinline__ bool insert_keys(K* tk, uint32_t mask, const K (&key)[U],
                                            uint32_t (&slot)[U], const bool (&ok)[U], bool (&fr)[U]) {
  constexpr K EMPTY = K(~K(0));
  auto cas = [&](uint32_t s, K k) -> K {
    if constexpr (sizeof(K) == 8) return lds_cas64(reinterpret_cast<u64*>(tk) + s, EMPTY64, k);
    else return lds_cas32(reinterpret_cast<uint32_t*>(tk) + s, EMPTY32, k);
  };
  K old[U];
  bool todo[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    old[u] = key[u];
    if (ok[u]) old[u] = cas(slot[u], key[u]);
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    fr[u] = ok[u] && old[u] == EMPTY;
    todo[u] = ok[u] && old[u] != EMPTY && old[u] != key[u];
  }
  for (uint32_t probe = 1; probe < NSGC_MAX_PROBES; ++probe) {
    u64 any = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) any |= __ballot(todo[u]);
    if (any == 0) break;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (todo[u]) {
        slot[u] = (slot[u] + probe_step(key[u])) & mask;
        old[u] = cas(slot[u], key[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      fr[u] = fr[u] || (todo[u] && old[u] == EMPTY);
      todo[u] = todo[u] && old[u] != EMPTY && old[u] != key[u];
    }
  }
  bool failed = false;
#pragma unroll
  for (int u = 0; u < U; ++u) failed = failed || todo[u];
  return failed;
}

constexpr uint32_t NO_SLOT = 0xFFFFFFFFu;

// Home slot of a link, from low bits that its cell leaves free (shifted, so that
// links of an address with itself spread where both views hash alike).
__device__ __forceinline__ uint32_t link_home(u64 k) { return uint32_t(k >> 32) ^ (uint32_t(k) >> 1); }

// Work queue of phases B and C: like ItemQueue, but the item after the next is
// requested as soon as the next one is announced, so that the answer is in
// before the item's stores go out (memory operations complete in order: a
// wait for it behind them would wait for them too).
struct GridQueue {
  NSGC_GLOBAL uint32_t* counter;
  uint32_t base, step, pending;   // pending: thread 0's requested position
  __device__ GridQueue(NSGC_GLOBAL uint32_t* counters, uint32_t items) {
    step = min(uint32_t(NSGC_QCLASSES), gridDim.x);
    const uint32_t c = blockIdx.x % step;
    counter = counters + c * NSGC_QSTRIDE;
    base = gridDim.x + c;          // after the grid's static first items
    pending = NO_ITEM;
    if (threadIdx.x == 0 && gridDim.x < items) take();   // (else each workgroup takes one item)
  }
  __device__ __forceinline__ void take() {
    pending = base + step * __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
  }
  // Thread 0 writes the next item (or NO_ITEM) to the LDS word *at and
  // requests the one after it; visible after the caller's next barrier.
  __device__ __forceinline__ void announce(uint32_t* at, uint32_t items) {
    if (threadIdx.x == 0) {
      *at = pending < items ? pending : NO_ITEM;
      if (pending < items) take();
    }
  }
};

// The value, arrived: a load the compiler has already seen waited for is not
// waited for again behind later stores.
template <class T>
__device__ __forceinline__ void arrived(T& x) {
  asm volatile("" : "+v"(x));
}
__device__ __forceinline__ void loads_arrived() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

}  // namespace

// ---------------------------------------------------------------------------
// Dominant addresses.  One workgroup per window counts the hashed sources
// (first half of its threads) and destinations (second half) of a sample of
// 2048 packets (4096 in batches with windows of more than 1024 cells), 64 runs
// spread from the window's first packet to its last.  An address is a
// candidate when the sample puts more than an eighth of a strip's share of the
// packets on it, or half a bucket's (and at least 8 hits); of two candidates
// that share an entry of the lookup table the more frequent one stays, and of
// those the most frequent NSGC_GRID_HEAVY.  The lookup's shift is the one of
// eight that leaves out the fewest hits: with a fixed one about four of 64
// addresses were left out, now and then a very frequent one, whose strip then
// overfilled (128 skewed windows of 2^23 packets 10.1 -> 9.6 ms).  The matrix
// starts at zero.  One trip to memory and a dozen barriers: bound by latency,
// 5 us for one window and 8.7 us for 64.
// ---------------------------------------------------------------------------

constexpr uint32_t GH_NT = 1024;
constexpr uint32_t GH_VT = GH_NT / 2;                       // threads per view
constexpr uint32_t GH_MIN = 8;                              // hits of a candidate
static_assert(HT == GH_VT, "one thread per table entry and per candidate");

template <uint32_t HV>
__global__ __launch_bounds__(GH_NT) void k_grid_heavy(const nsgc_dev_plan* __restrict__ P) {
  constexpr uint32_t SAMPLE = NSGC_GRID_SAMPLE(HV);
  constexpr uint32_t GH_PER = SAMPLE / GH_VT;      // sampled packets per thread
  constexpr uint32_t GH_TABLE = 2 * SAMPLE;
  constexpr uint32_t GH_CAND = SAMPLE / GH_MIN;    // at most so many candidates per view
  constexpr uint32_t RUN = SAMPLE / 64;
  static_assert(GH_CAND <= GH_VT && HEAVY_SHIFTS * HT * 8 <= 2 * GH_TABLE * 4, "entries lie in the table");
  __shared__ __align__(16) uint32_t table[2][2][GH_TABLE];   // ids and counts of each view
  __shared__ u64 cand[2][GH_CAND];            // hits << 32 | id
  __shared__ uint32_t lost[2][HEAVY_SHIFTS];   // hits of the candidates without an entry
  __shared__ uint32_t ncand[2];
  const uint32_t v = threadIdx.x >= GH_VT ? 1u : 0u;   // view: sources, destinations
  const ColHash dst_hash(P->entity != 0);
  const uint32_t tid = threadIdx.x & (GH_VT - 1);
  uint32_t* const k = table[v][0];
  uint32_t* const c = table[v][1];
  for (uint32_t wi = blockIdx.x; wi < P->num_grid; wi += gridDim.x) {
    const nsgc_grid_desc W = sload_words(P->gwin + wi);
    const NSGC_GLOBAL uint32_t* col = gptr(v ? W.dst : W.src);
    uint32_t x[GH_PER];
#pragma unroll
    for (uint32_t u = 0; u < GH_PER; ++u) {
      const uint32_t s = u * GH_VT + tid;
      x[u] = col[uint32_t(u64(W.n - RUN) * (s / RUN) / 63u) + s % RUN];
    }
    const v4u32 e4 = {EMPTY32, EMPTY32, EMPTY32, EMPTY32}, z4 = {0u, 0u, 0u, 0u};
#pragma unroll
    for (uint32_t i = 0; i < GH_TABLE / 4 / GH_VT; ++i) {
      reinterpret_cast<v4u32*>(k)[i * GH_VT + tid] = e4;
      reinterpret_cast<v4u32*>(c)[i * GH_VT + tid] = z4;
    }
    if (tid == 0) ncand[v] = 0;
    if (tid < HEAVY_SHIFTS) lost[v][tid] = 0;
    NSGC_GLOBAL uint32_t* out = gptr(W.heavy);
    for (uint32_t i = threadIdx.x; i < HV * HV; i += GH_NT) out[2 * HV + i] = 0;
    if (threadIdx.x < 2 * HV) out[threadIdx.x] = EMPTY32;   // unused (this id is never dominant)
    lds_barrier();
#pragma unroll
    for (uint32_t u = 0; u < GH_PER; ++u) {
      const uint32_t id = v ? dst_hash(x[u]) : row_hash(x[u]);
      if (id == EMPTY32) continue;   // the tables' marker keeps its own path
      uint32_t sl = id & (GH_TABLE - 1);
      for (;;) {   // ends: the table holds twice the sample
        const uint32_t old = lds_cas32(k + sl, EMPTY32, id);
        if (old == EMPTY32 || old == id) break;
        sl = (sl + 1) & (GH_TABLE - 1);
      }
      lds_add(&c[sl], 1);
    }
    lds_barrier();
    const uint32_t strip = v ? W.logBc : W.logA, bucket = v ? W.logC : W.logR;
    const uint32_t thr = max(GH_MIN, min(SAMPLE >> (strip + 3), SAMPLE >> (bucket + 1)));
#pragma unroll
    for (uint32_t i = 0; i < GH_TABLE / GH_VT; ++i) {
      const uint32_t h = c[i * GH_VT + tid];
      if (h >= thr) cand[v][lds_add(&ncand[v], 1)] = (u64(h) << 32) | k[i * GH_VT + tid];
    }
    lds_barrier();
    // the candidate that holds each entry under each shift, where the table was
    u64* const best = reinterpret_cast<u64*>(k);
#pragma unroll
    for (uint32_t i = 0; i < HEAVY_SHIFTS; ++i) best[i * HT + tid] = 0;
    lds_barrier();
    u64 mine = tid < ncand[v] ? cand[v][tid] : 0ull;
    if (mine) {
#pragma unroll
      for (uint32_t i = 0; i < HEAVY_SHIFTS; ++i)
        __hip_atomic_fetch_max(&best[i * HT + heavy_index(uint32_t(mine), i)], mine, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    lds_barrier();
    if (mine) {
#pragma unroll
      for (uint32_t i = 0; i < HEAVY_SHIFTS; ++i)
        if (best[i * HT + heavy_index(uint32_t(mine), i)] != mine) lds_add(&lost[v][i], uint32_t(mine >> 32));
    }
    lds_barrier();
    uint32_t shift = 0;
#pragma unroll
    for (uint32_t i = 1; i < HEAVY_SHIFTS; ++i)
      if (lost[v][i] < lost[v][shift]) shift = i;
    if (tid == 0) out[2 * HV + HV * HV + v] = shift;
    if (mine && best[shift * HT + heavy_index(uint32_t(mine), shift)] != mine) mine = 0;
    __syncthreads();   // (the unused marks in memory land before the ids below)
    if (tid < GH_CAND && !mine) cand[v][tid] = 0;
    lds_barrier();
    if (mine) {
      uint32_t rank = 0;
      const uint32_t nc = ncand[v];
      for (uint32_t i = 0; i < nc; ++i) rank += cand[v][i] > mine;
      if (rank < HV) out[v * HV + rank] = uint32_t(mine);
    }
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// Phase A: a tile's packets ordered by cell.  Each workgroup takes a
// contiguous run of tiles, so that it adds its part of a window's dominant
// matrix to memory once per window and not once per tile.  The next tile's
// packets are loaded while the current one's keys are written.  Moves 8 bytes
// per packet in and up to 8 out: 2^23 packets (64 windows) in 37 us, 2^30 (128
// windows, 2048 cells) in 3.8 ms, 3.4 TB/s of the copy rate's 5.1; LDS counting
// and placing, one workgroup of 1024 per compute unit, is the rest.
// ---------------------------------------------------------------------------

namespace {
constexpr size_t grid_part_lds(uint32_t tile_log2, uint32_t cells) {
  const size_t HV = size_t(NSGC_GRID_HV(tile_log2));
  return (size_t(1) << tile_log2) * 8 + (cells + 4) * 4 + HV * HV * 4 + 2 * HT * 4 + 2 * HT + 64;
}
}  // namespace

size_t lds_grid_part_bytes(uint32_t tile_log2, uint32_t max_cells) {
  return grid_part_lds(tile_log2, max_cells);
}

// KEYS: the window's packets are link keys already (W.src points to them).
template <int PER, int NT, uint32_t HV, bool KEYS = false>
__global__ __launch_bounds__(NT) void k_grid_partition(const nsgc_dev_plan* __restrict__ P,
                                                       uint32_t max_cells) {
  static_assert(PER % 4 == 0, "PER must be a multiple of 4");
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr uint32_t T = NT * PER;
  constexpr int NW = NT / 64;
  u64* stage = reinterpret_cast<u64*>(smem);                       // [T]
  uint32_t* hist = reinterpret_cast<uint32_t*>(stage + T);         // [max_cells + 1]
  uint32_t* mat = hist + max_cells + 4;                            // [HV][HV]
  uint32_t* idt = mat + HV * HV;                                   // [2][HT] dominant ids
  uint8_t* ids = reinterpret_cast<uint8_t*>(idt + 2 * HT);         // [2][HT] their slots
  uint32_t* red = reinterpret_cast<uint32_t*>(ids + 2 * HT);       // [NW]
  const uint32_t tid = threadIdx.x, w = tid >> 6;
  const ColHash dst_hash(sload(&P->entity) != 0);
  const uint32_t items = P->gitemsA;
  const uint32_t per = (items + gridDim.x - 1) / gridDim.x;
  const uint32_t beg = min(items, blockIdx.x * per), end = min(items, beg + per);
  if (beg >= end) return;
  uint32_t wi = uniform(owner_of_wave(gptr(P->gprefA), P->num_grid, beg));
  nsgc_grid_desc W = sload_words(P->gwin + wi);
  uint32_t first = sload(P->gprefA + wi), next = sload(P->gprefA + wi + 1);

  // The window's dominant ids into the lookup table (a free entry holds an id
  // that belongs to another entry).  Needs a barrier before and after.
  uint32_t sh = 0, dh = 0;   // lookup shifts
  auto load_heavy = [&]() {
    sh = uniform(gptr(W.heavy)[2 * HV + HV * HV]);
    dh = uniform(gptr(W.heavy)[2 * HV + HV * HV + 1]);
    for (uint32_t i = tid; i < 2 * HT; i += NT) idt[i] = free_entry(i, i < HT ? sh : dh);
    lds_barrier();
    if (tid < 2 * HV) {
      const uint32_t id = gptr(W.heavy)[tid];
      if (id != EMPTY32) {
        const uint32_t at = (tid / HV) * HT + heavy_index(id, tid < HV ? sh : dh);
        idt[at] = id;
        ids[at] = uint8_t(tid & (HV - 1));
      }
    }
  };
  auto flush = [&]() {   // the matrix counted so far to memory; leaves it zero
    NSGC_GLOBAL uint32_t* m = gptr(W.heavy) + 2 * HV;
    for (uint32_t i = tid; i < HV * HV; i += NT) {
      if (mat[i]) __hip_atomic_fetch_add(m + i, mat[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      mat[i] = 0;
    }
  };
  uint32_t r[PER], c[PER];
  auto load = [&](uint32_t tbeg, uint32_t len) {
    if constexpr (KEYS) {
      const NSGC_GLOBAL u64* in = (const NSGC_GLOBAL u64*)gptr(W.src) + tbeg;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const u64 x = in[min(uint32_t((k >> 2) * NT + tid) * 4 + (k & 3), len - 1)];
        r[k] = uint32_t(x >> 32);
        c[k] = uint32_t(x);
      }
      return;
    }
    const NSGC_GLOBAL uint32_t* src = gptr(W.src) + tbeg;
    const NSGC_GLOBAL uint32_t* dst = gptr(W.dst) + tbeg;
    if (len == T) {
#pragma unroll
      for (int k = 0; k < PER / 4; ++k) {
        const uint32_t idx = (k * NT + tid) * 4;
        const v4u32 s4 = *(const NSGC_GLOBAL v4u32_any*)(src + idx);
        const v4u32 d4 = *(const NSGC_GLOBAL v4u32_any*)(dst + idx);
        r[4 * k + 0] = s4.x; r[4 * k + 1] = s4.y; r[4 * k + 2] = s4.z; r[4 * k + 3] = s4.w;
        c[4 * k + 0] = d4.x; c[4 * k + 1] = d4.y; c[4 * k + 2] = d4.z; c[4 * k + 3] = d4.w;
      }
    } else {   // a window's last tile: a packet past the end repeats the last one, masked below
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const uint32_t at = min(uint32_t((k >> 2) * NT + tid) * 4 + (k & 3), len - 1);
        r[k] = src[at];
        c[k] = dst[at];
      }
    }
  };

  uint32_t t = beg - first, len = min(T, W.n - t * T);
  load(t * T, len);
  for (uint32_t i = tid; i < HV * HV; i += NT) mat[i] = 0;
  load_heavy();
  for (uint32_t item = beg;; ++item) {
    const uint32_t a = W.logA, b = W.logBc, cells = 1u << (W.subA + W.subB);
    for (uint32_t i = tid; i < cells; i += NT) hist[i] = 0;
    lds_barrier();
    uint32_t br[PER];   // rank in cell << 12 | cell; all ones: no key
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if constexpr (!KEYS) {
        r[k] = row_hash(r[k]);
        c[k] = dst_hash(c[k]);
      }
      const bool hs = idt[heavy_index(r[k], sh)] == r[k], hd = idt[HT + heavy_index(c[k], dh)] == c[k];
      const bool ok = len == T || uint32_t((k >> 2) * NT + tid) * 4 + (k & 3) < len;
      br[k] = ~0u;
      uint32_t i = r[k] >> (32 - a), j = c[k] >> (32 - b);
      if (hs && hd) {
        if (ok) lds_add(&mat[uint32_t(ids[heavy_index(r[k], sh)]) * HV + ids[HT + heavy_index(c[k], dh)]], 1);
      } else {
        // a key names a dominant address by its slot, off the cell's strip
        if (hs) {
          i ^= strip_shift(c[k], a);
          r[k] = ((i ^ 1u) << (32 - a)) | ids[heavy_index(r[k], sh)];
        }
        if (hd) {
          j ^= strip_shift(r[k], b);
          c[k] = ((j ^ 1u) << (32 - b)) | ids[HT + heavy_index(c[k], dh)];
        }
        const uint32_t cell = ((i & ((1u << W.subA) - 1u)) << W.subB) | (j & ((1u << W.subB) - 1u));
        if (ok) br[k] = (lds_add(&hist[cell], 1) << 12) | cell;
      }
    }
    lds_barrier();
    // counts -> starts
    {
      const uint32_t q = (cells + NT - 1) / NT;
      const uint32_t h0 = min(cells, tid * q), h1 = min(cells, h0 + q);
      uint32_t s = 0;
      for (uint32_t i = h0; i < h1; ++i) s += hist[i];
      const uint32_t incl = wave_inclusive_scan(s);
      if (lane_id() == 63) red[w] = incl;
      lds_barrier();
      uint32_t run = incl - s, all = 0;
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const uint32_t x = red[k];
        if (uint32_t(k) < w) run += x;
        all += x;
      }
      // the tile records go out here, start | length << 16
      NSGC_GLOBAL uint32_t* tm = gptr(W.tile) + u64(t) * cells;
      for (uint32_t i = h0; i < h1; ++i) {
        const uint32_t x = hist[i];
        hist[i] = run;
        tm[i] = run | (x << 16);
        run += x;
      }
      if (tid == 0) hist[cells] = all;
    }
    lds_barrier();
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (br[k] != ~0u) stage[hist[br[k] & 0xFFFu] + (br[k] >> 12)] = (u64(r[k]) << 32) | c[k];
    const uint32_t total = hist[cells];
    NSGC_GLOBAL u64* out = gptr(W.keys) + t * T;
    lds_barrier();
    const bool more = item + 1 < end;
    if (more) {
      if (item + 1 >= next) {   // the run goes on into another window
        flush();
        do {
          first = next;
          next = sload(P->gprefA + ++wi + 1);
        } while (item + 1 >= next);
        W = sload_words(P->gwin + wi);
        load_heavy();
      }
      t = item + 1 - first;
      len = min(T, W.n - t * T);
      load(t * T, len);
    }
    for (uint32_t i = tid; i < total; i += NT) out[i] = stage[i];
    if (!more) break;
  }
  lds_barrier();
  flush();
}

// ---------------------------------------------------------------------------
// Shared by phases B and C: the elements of a list of segments, spread over
// the workgroup.  Thread s describes segment s (n <= NT segments: base, len);
// on return list[e] is the position of element e of their concatenation, for
// all e below the total (returned; nothing is written if it exceeds `room`).
// Groups of 2^g threads walk one segment each, as many as NT / n allows.
// `tab` is LDS scratch of 2 * NT + 2 * NT / 64 words.  Begins and ends with
// work that needs the caller's barrier: the caller passes one before `list`
// and `tab` may be written and one before `list` is read.
// ---------------------------------------------------------------------------

template <int NT>
__device__ __forceinline__ uint32_t spread_segments(uint32_t tid, uint32_t n, uint32_t base, uint32_t len,
                                                    uint32_t& extra, uint32_t* tab, uint32_t* list,
                                                    uint32_t room) {
  constexpr int NW = NT / 64;
  const uint32_t w = tid >> 6;
  uint32_t* start = tab;
  uint32_t* pos = tab + NT;
  uint32_t* red = tab + 2 * NT;
  const uint32_t incl = wave_inclusive_scan(len);
  const uint32_t ex = wave_sum(extra);
  if (lane_id() == 63) {
    red[w] = incl;
    red[NW + w] = ex;
  }
  pos[tid] = base;
  lds_barrier();
  uint32_t before = 0, total = 0, xs = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    const uint32_t x = red[k];
    if (uint32_t(k) < w) before += x;
    total += x;
    xs += red[NW + k];
  }
  extra = uniform(xs);
  total = uniform(total);
  if (total > room) return total;
  start[tid] = before + incl - len;
  lds_barrier();
  const uint32_t lg = min(6u, 31u - uint32_t(__builtin_clz(uint32_t(NT) / max(n, 1u))));
  const uint32_t s = tid >> lg, g = 1u << lg;
  if (s < n) {
    const uint32_t at = start[s], p = pos[s];
    const uint32_t l = (s + 1 < n ? start[s + 1] : total) - at;
    for (uint32_t k = tid & (g - 1); k < l; k += g) list[at + k] = p + k;
  }
  return total;
}

// The same for at most 64 segments, described alike in every wavefront (lane
// s: segment s): no barrier inside.
template <int NT>
__device__ __forceinline__ uint32_t spread_by_wave(uint32_t tid, uint32_t n, uint32_t base, uint32_t len,
                                                   uint32_t& extra, uint32_t* list, uint32_t room) {
  const uint32_t incl = wave_inclusive_scan(len);
  const uint32_t total = uniform(readlane(incl, 63));
  extra = uniform(wave_sum(extra));
  if (total > room) return total;
  const uint32_t lg = 31u - uint32_t(__builtin_clz(uint32_t(NT) / max(n, 1u)));
  const uint32_t s = tid >> lg, g = 1u << lg;
  const uint32_t at = lane_take(incl - len, s), p = lane_take(base, s), l = lane_take(len, s);
  if (s < n)
    for (uint32_t k = tid & (g - 1); k < l; k += g) list[at + k] = p + k;
  return total;
}

// ---------------------------------------------------------------------------
// Phase B: the links of one cell.  Bound by the latency of the item's serial
// chain (records, positions, keys, table, counts, starts, stores), hidden by
// five (BIG: three) workgroups per compute unit and by loading the next item's
// records and asking for the one after it during the current one.  Keys stay in
// registers from the insert to the emission: reading them again, or the table,
// is another trip through LDS for every slot.  64 windows of 2^17 packets in 76
// us against 94 us with a wavefront per link bucket; 128 of 2^23 in 3.8 ms
// against 8.4 ms with a workgroup per link bucket.  Measured and not taken: all
// four home slots probing on in step (88 us), entries staged in LDS and copied
// out in lines (83 us), cells twice the size (100 us).
// ---------------------------------------------------------------------------

// The table, the CW words of counts, the bins and the flags of a cell, empty.
template <int NT, int SL, int CW>
__device__ __forceinline__ void clear_cell_table(uint32_t tid, u64* tk, uint32_t* tc, uint32_t* bin,
                                                 uint32_t* misc) {
  const v4u32 e4 = {EMPTY32, EMPTY32, EMPTY32, EMPTY32}, z4 = {0u, 0u, 0u, 0u};
#pragma unroll
  for (uint32_t i = 0; i < SL / 2 / NT; ++i) reinterpret_cast<v4u32*>(tk)[i * NT + tid] = e4;
#pragma unroll
  for (uint32_t i = 0; i < CW / 4 / NT; ++i) reinterpret_cast<v4u32*>(tc)[i * NT + tid] = z4;
  if (tid < 2 * NSGC_GRID_MAX_SUB) bin[tid] = 0;
  if (tid < 4) misc[tid] = 0;
}

// Counts -> exclusive starts of the row and the column bins: every wavefront
// scans both (at most 64 bins, one per lane; lane i returns bin i's starts);
// the first one publishes them for phase C.
__device__ __forceinline__ void publish_starts(NSGC_GLOBAL uint32_t* rec, const uint32_t* bin,
                                               uint32_t rsub, uint32_t csub, uint32_t below,
                                               uint32_t& xr, uint32_t& xc) {
  const uint32_t lane = lane_id();
  const uint32_t nr = lane < rsub ? bin[lane] : 0u;
  const uint32_t nc = lane < csub ? bin[NSGC_GRID_MAX_SUB + lane] : 0u;
  const uint32_t ir = wave_inclusive_scan(nr), ic = wave_inclusive_scan(nc);
  xr = ir - nr;
  xc = ic - nc;
  if (threadIdx.x < 64) {
    if (lane == 0) rec[0] = below;
    if (lane < rsub) rec[1 + lane] = xr;
    if (lane < csub) rec[2 + rsub + lane] = xc;
    if (lane == 63) {
      rec[1 + rsub] = ir;
      rec[2 + rsub + csub] = ic;
    }
  }
}

// ---------------------------------------------------------------------------
// The cells that are too large for the single passes (more keys than their
// threads hold, or more links than their tables take), a workgroup each.
//
// By rounds: each fills the table with as many links as it takes, which are
// counted, emitted and overwritten with the marker, so that the next round sees
// only the others.  A round reads the cell's keys twice, so a cell of k links
// costs 2 k / GR_FULL readings: the cells that are left over in ordinary traffic
// have a few thousand to a few tens of thousands.  A cell of more than GR_KEYS
// keys, or whose table was full after less than one key in GR_ROUNDS, is sorted
// instead: eight passes over its keys whatever they are (cells are chosen by the
// top bits of the hashed addresses, so traffic can be made that puts a whole
// window in one).  Sorting 2^16 keys takes as long as three or four rounds, but
// links that repeat need fewer rounds than the first one lets expect.
// One workgroup of 1024 threads with 8192 slots per compute unit: against two of
// 512 with 4096, one window of 2^26 packets among 4096 addresses (8192 links in
// each cell) takes 3.8 ms instead of 6.2, one of 2^25 2.3 instead of 3.2.
// ---------------------------------------------------------------------------

constexpr int GR_NT = 1024;
constexpr int GR_SL = 8192;
constexpr uint32_t GR_FULL = GR_SL * 3 / 4;   // links in the table when no more are taken
constexpr uint32_t GR_ROUNDS = 6;
constexpr uint32_t GR_KEYS = 1u << 16;

// The n keys that `each` visits (in any order) into `a` in ascending order, by way of `b`: a radix sort by bytes.
// `lds` is scratch of 2048 + 4 NT words.  Ends with a barrier.
template <int NT, class Each>
__device__ __forceinline__ void sort_cell(uint32_t n, NSGC_GLOBAL u64* a, NSGC_GLOBAL u64* b, uint32_t* lds,
                                          const Each& each) {
  constexpr uint32_t NW = NT / 64, R = 8, TILE = NT * R;
  static_assert(NW >= 8, "a wavefront per digit scans its counts");
  uint32_t* const hist = lds;          // [8][256] of each digit: counts, then the next position
  uint32_t* const cnt = lds + 2048;    // [NW][256]
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = lane_id();
  auto digit = [](u64 k, uint32_t d) { return uint32_t(k >> (8 * d)) & 255u; };
  __syncthreads();
  for (uint32_t i = tid; i < 2048; i += NT) hist[i] = 0;
  __syncthreads();
  each([&](u64 k) {
#pragma unroll
    for (uint32_t d = 0; d < 8; ++d) lds_add(&hist[d * 256 + digit(k, d)], 1);
  });
  __syncthreads();
  if (w < 8) {
    uint32_t x[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = s;
      s += hist[w * 256 + lane * 4 + k];
    }
    const uint32_t before = wave_inclusive_scan(s) - s;
#pragma unroll
    for (int k = 0; k < 4; ++k) hist[w * 256 + lane * 4 + k] = before + x[k];
  }
  __syncthreads();
  each([&](u64 k) { b[lds_add(&hist[digit(k, 0)], 1)] = k; });   // (any order within a digit)
  __syncthreads();
  for (uint32_t d = 1; d < 8; ++d) {
    const NSGC_GLOBAL u64* in = d & 1u ? b : a;
    NSGC_GLOBAL u64* out = d & 1u ? a : b;
    uint32_t pos = hist[d * 256 + (tid & 255u)];   // of digit `tid`, as it runs through the tiles
    for (uint32_t base = 0; base < n; base += min(TILE, n - base)) {
      for (uint32_t i = lane; i < 256; i += 64) cnt[w * 256 + i] = 0;
      const uint32_t len = min(TILE, n - base), w0 = w * (R * 64) + lane;
      u64 key[R];
      uint32_t rk[R];
#pragma unroll
      for (uint32_t r = 0; r < R; ++r) key[r] = w0 + r * 64 < len ? in[base + w0 + r * 64] : 0ull;
#pragma unroll
      for (uint32_t r = 0; r < R; ++r) {   // rank among the wavefront's keys with this digit, in order
        const bool ok = w0 + r * 64 < len;
        const uint32_t x = digit(key[r], d);
        u64 m = __ballot(ok);
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
          const u64 mb = __ballot((x >> k) & 1u);
          m &= ((x >> k) & 1u) ? mb : ~mb;
        }
        const uint32_t leader = ok ? uint32_t(__ffsll(static_cast<unsigned long long>(m)) - 1) : 0u;
        uint32_t old = 0;
        if (ok && lane == leader) old = lds_add(&cnt[w * 256 + x], uint32_t(__popcll(m)));
        rk[r] = lane_take(old, leader) + rank_below(m);
      }
      __syncthreads();
      if (tid < 256) {
#pragma unroll
        for (uint32_t k = 0; k < NW; ++k) {
          const uint32_t c = cnt[k * 256 + tid];
          cnt[k * 256 + tid] = pos;
          pos += c;
        }
      }
      __syncthreads();
#pragma unroll
      for (uint32_t r = 0; r < R; ++r)
        if (w0 + r * 64 < len) out[cnt[w * 256 + digit(key[r], d)] + rk[r]] = key[r];
      __syncthreads();
    }
  }
}

// Visits the runs of equal keys of the sorted a[0 .. n), n >= 1: fn(key, length),
// by the thread that meets a run's last key.  When it is called, every thread has
// read all keys up to that one (and those of later runs up to the end of its 512
// are in registers), so it may write where they were.  `lds` is scratch of 2 * NT
// / 64 words.  Begins and ends with a barrier.
template <int NT, class Fn>
__device__ __forceinline__ void sorted_runs(uint32_t n, const NSGC_GLOBAL u64* a, uint32_t* lds, const Fn& fn) {
  constexpr uint32_t NW = NT / 64;
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = lane_id();
  uint32_t carry = 0, side = 0;   // start of the run that the next keys belong to
  __syncthreads();
  for (uint32_t base = 0; base < n; base += min(uint32_t(NT), n - base)) {
    const uint32_t left = n - base, i = min(tid, left - 1u);
    const u64 key = a[base + i], next = a[base + min(i + 1u, left - 1u)];
    const bool end = tid < left && (tid + 1u == left || next != key);
    const u64 m = __ballot(end);
    uint32_t* const after = lds + side * NW;   // key after the wavefront's last run, 0 if none ends in it
    if (lane == 0) after[w] = m ? base + w * 64 + 64u - uint32_t(__clzll(static_cast<long long>(m))) : 0u;
    __syncthreads();
    uint32_t start = carry;
#pragma unroll
    for (uint32_t k = 0; k < NW; ++k) {
      const uint32_t x = after[k];
      if (k < w) start = max(start, x);
      carry = max(carry, x);
    }
    const u64 mine = m & ((u64(1) << lane) - 1u);
    if (mine) start = base + w * 64 + 64u - uint32_t(__clzll(static_cast<long long>(mine)));
    if (end) fn(key, base + tid + 1u - start);
    side ^= 1u;
  }
  __syncthreads();
}

__global__ __launch_bounds__(GR_NT) void k_grid_rounds(nsgc_dev_plan* P, uint32_t after_wide) {
  constexpr int NT = GR_NT, SL = GR_SL, NW = NT / 64;
  __shared__ __align__(16) u64 tk[SL];
  __shared__ __align__(16) uint32_t tc[SL];
  __shared__ u64 acc[2 * HVM];
  __shared__ uint32_t bin[2 * NSGC_GRID_MAX_SUB];   // rows, columns
  __shared__ uint32_t misc[4];   // 0 failed, 1 special packets, 2 links, 3 max packets
  __shared__ uint32_t fill[3];   // of a round: links in the table, keys read by then, keys left over
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t items = P->gover[after_wide ? 2 : 0];
  for (uint32_t x = blockIdx.x; x < items; x += gridDim.x) {
  const uint32_t it = uniform(gptr(after_wide ? sload(&P->goverW) : sload(&P->goverB))[x]);
  const uint32_t HV = NSGC_GRID_HV(sload(&P->gtile_log2));
  if (tid < 2 * HV) acc[tid] = 0;
  const uint32_t T = 1u << sload(&P->gtile_log2);
  const nsgc_grid_desc W = sload_words(sload(&P->gwin) + sload(sload(&P->gitemB) + it));
  const uint32_t cell = it - W.itemB;
  const uint32_t a = W.logA, b = W.logBc, cells = 1u << (W.subA + W.subB);
  const uint32_t ci = W.strip_i + (cell >> W.subB), cj = W.strip_j + (cell & ((1u << W.subB) - 1u));
  const uint32_t rsub = 1u << (W.logR - a), csub = 1u << (W.logC - b);
  const uint32_t nt = W.ntiles;
  NSGC_GLOBAL u64* keys = gptr(W.keys);
  const NSGC_GLOBAL uint32_t* tm = gptr(W.tile) + cell;
  NSGC_GLOBAL uint32_t* rec = gptr(W.rec) + u64(cell) * (rsub + csub + 3);
  uint32_t below = 0, total = 0;   // keys of the window in cells below this one; its own
  for (uint32_t t = tid; t < nt; t += NT) {
    const uint32_t y = tm[u64(t) * cells];
    below += y & 0xFFFFu;
    total += y >> 16;
  }
  below = wave_sum(below);
  total = wave_sum(total);
  if (lane == 0) {
    tc[tid >> 6] = below;
    tc[NW + (tid >> 6)] = total;
  }
  __syncthreads();
  below = total = 0;
  for (int k = 0; k < NW; ++k) {
    below += tc[k];
    total += tc[NW + k];
  }
  below = uniform(below);
  total = uniform(total);
  NSGC_GLOBAL u64* er = gptr(W.emit_row) + W.base + below;
  NSGC_GLOBAL u64* ec = gptr(W.emit_col) + W.base + below;
  auto row_bin = [&](uint32_t r) { return (r >> (32 - W.logR)) & (rsub - 1u); };
  auto col_bin = [&](uint32_t c) { return (c >> (32 - W.logC)) & (csub - 1u); };
  auto row_light = [&](uint32_t r) { return (r >> (32 - a)) == ci; };
  auto col_light = [&](uint32_t c) { return (c >> (32 - b)) == cj; };
  auto home = [&](u64 k) { return link_home(k) & uint32_t(SL - 1); };
  auto add_heavy = [&](uint32_t v, uint32_t id, uint32_t n) {
    lds_add64(&acc[v * HV + (id & (HV - 1))], (u64(1) << 32) | n);
  };
  auto clear_table = [&]() { clear_cell_table<NT, SL, SL>(tid, tk, tc, bin, misc); };
  // The bins' counts to starts, published and left in `bin` as emission cursors.
  auto starts = [&]() {
    __syncthreads();
    uint32_t xr, xc;
    publish_starts(rec, bin, rsub, csub, W.base + below, xr, xc);
    __syncthreads();
    if (tid < 64) {
      if (lane < rsub) bin[lane] = xr;
      if (lane < csub) bin[NSGC_GRID_MAX_SUB + lane] = xc;
    }
    __syncthreads();
  };
  auto emit_row = [&](uint32_t r, uint32_t n) {
    const uint32_t parts = entry_parts(n, 1);
    if (row_light(r)) write_entry(er, lds_add(&bin[row_bin(r)], parts), r, n, 1, parts);
  };
  auto emit_col = [&](uint32_t c, uint32_t n) {
    const uint32_t parts = entry_parts(n, 1);
    if (col_light(c)) write_entry(ec, lds_add(&bin[NSGC_GRID_MAX_SUB + col_bin(c)], parts), c, n, 1, parts);
  };

  uint32_t links = 0, mx = 0;
  const uint32_t most = sload(&P->gmax_keys);
  bool abandoned = most && total / 16 > most;
  uint32_t special = 0;
  const uint32_t max_rounds = 1u << min(sload(&P->max_sweeps_log2), 24u);
  auto seg = [&](uint32_t t, u64& base, uint32_t& len) {
    const uint32_t x = tm[u64(t) * cells];
    base = u64(t) * T + (x & 0xFFFFu);
    len = x >> 16;
  };
  for (uint32_t round = 0; !abandoned; ++round) {
    if (round >= max_rounds) { abandoned = true; break; }
    __syncthreads();
    const uint32_t keep = round && tid < 2 * NSGC_GRID_MAX_SUB ? bin[tid] : 0u;
    clear_table();
    if (tid < 3) fill[tid] = 0;
    if (round && tid < 2 * NSGC_GRID_MAX_SUB) bin[tid] = keep;   // cursors stay
    __syncthreads();
    gather_by_wave<4, NW>(nt, seg, [&](const auto& pos, const auto& okin) {
      constexpr int U = array_len<decltype(pos)>();
      if (lds_load(&misc[0])) return;   // the table takes no more
      u64 key[U];
      uint32_t at[U], add[U];
      bool ok[U], fr[U];
      uint32_t read = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) key[u] = keys[okin[u] ? pos[u] : 0ull];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        ok[u] = okin[u];
        at[u] = home(key[u]);
        add[u] = 1;
        if (ok[u] && key[u] == EMPTY64) {   // round 0: special; later: counted already
          if (round == 0) lds_add(&misc[1], 1);
          ok[u] = false;
        }
        // combine the lanes holding the first valid lane's key
        const u64 vm = __ballot(ok[u]);
        read += __popcll(vm);
        if (vm) {
          const int f = __ffsll(static_cast<unsigned long long>(vm)) - 1;
          const bool same = ok[u] && key[u] == readlane64(key[u], uint32_t(f));
          const uint32_t ns = __popcll(__ballot(same));
          if (ns > 1 && same) {
            if (int(lane_id()) == f) add[u] = ns;
            else ok[u] = false;
          }
        }
      }
      if (insert_keys<U>(tk, uint32_t(SL - 1), key, at, ok, fr)) lds_store(&misc[0], 1);
      uint32_t fresh = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (ok[u]) lds_add(&tc[at[u]], add[u]);   // (a failed round counts again, what the table holds)
        fresh += __popcll(__ballot(fr[u]));
      }
      if (lane_id() == 0) {
        lds_add(&fill[1], read);
        if (fresh && lds_add(&fill[0], fresh) + fresh > GR_FULL) lds_store(&misc[0], 1);
      }
    });
    const bool failed = misc[0] != 0;
    if (failed && round == 0 && (total > GR_KEYS || total > GR_ROUNDS * fill[1])) {
      // (it stands for GR_ROUNDS rounds where their number is limited)
      if (max_rounds <= GR_ROUNDS || (most && total > most)) { abandoned = true; break; }
      sort_cell<NT>(total, er, ec, reinterpret_cast<uint32_t*>(tk), [&](const auto& fn) {
        for (uint32_t t = uniform(tid >> 6); t < nt; t += NW) {
          u64 base;
          uint32_t len;
          seg(t, base, len);
          for (uint32_t i = lane; i < len; i += 64) fn(keys[base + i]);
        }
      });
      if (tid < 2 * NSGC_GRID_MAX_SUB) bin[tid] = 0;
      sorted_runs<NT>(total, er, tc, [&](u64 k, uint32_t n) {
        const uint32_t r = uint32_t(k >> 32), c = uint32_t(k), parts = entry_parts(n, 1);
        ++links;
        mx = max(mx, n);
        if (row_light(r)) lds_add(&bin[row_bin(r)], parts);
        else add_heavy(0, r, n);
        if (col_light(c)) lds_add(&bin[NSGC_GRID_MAX_SUB + col_bin(c)], parts);
        else add_heavy(1, c, n);
      });
      starts();
      // The row entries go where the keys were: the light sources' keys are
      // together and in the order of their bins, and a link has no more entries
      // than keys, so no entry lies behind the last key of its link.
      sorted_runs<NT>(total, er, tc, [&](u64 k, uint32_t n) {
        emit_row(uint32_t(k >> 32), n);
        emit_col(uint32_t(k), n);
      });
      break;
    }
    uint32_t left = 0;   // this thread's keys that found no place
    if (failed) {   // count the packets of the links that the table holds, and mark them
      for (uint32_t i = tid; i < SL; i += NT) tc[i] = 0;
      if (tid == 0) misc[1] = 0;
      __syncthreads();
      gather_by_wave<4, NW>(nt, seg, [&](const auto& pos, const auto& okin) {
        constexpr int U = array_len<decltype(pos)>();
        u64 key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = keys[okin[u] ? pos[u] : 0ull];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (!okin[u]) continue;
          if (round == 0) {   // a bin's segment: one slot per packet, the most entries it can receive
            if (row_light(uint32_t(key[u] >> 32))) lds_add(&bin[row_bin(uint32_t(key[u] >> 32))], 1);
            if (col_light(uint32_t(key[u]))) lds_add(&bin[NSGC_GRID_MAX_SUB + col_bin(uint32_t(key[u]))], 1);
          }
          if (key[u] == EMPTY64) {
            if (round == 0) lds_add(&misc[1], 1);
            continue;
          }
          uint32_t s = home(key[u]);
          u64 cur = tk[s];
          for (uint32_t p = 1; cur != key[u] && cur != EMPTY64 && p < NSGC_MAX_PROBES; ++p) {
            s = (s + probe_step(key[u])) & uint32_t(SL - 1);
            cur = tk[s];
          }
          if (cur == key[u]) {
            lds_add(&tc[s], 1);
            keys[pos[u]] = EMPTY64;
          } else {
            ++left;
          }
        }
      });
      left = wave_sum(left);
      if (lane == 0 && left) lds_add(&fill[2], left);
    } else if (round == 0) {   // everything fits: count the entries per bin
      for (uint32_t s = tid; s < SL; s += NT) {
        const u64 k = tk[s];
        if (k == EMPTY64) continue;
        const uint32_t parts = entry_parts(tc[s], 1);
        if (row_light(uint32_t(k >> 32))) lds_add(&bin[row_bin(uint32_t(k >> 32))], parts);
        if (col_light(uint32_t(k))) lds_add(&bin[NSGC_GRID_MAX_SUB + col_bin(uint32_t(k))], parts);
      }
      if (tid == 0 && misc[1]) {
        const uint32_t parts = entry_parts(misc[1], 1);
        lds_add(&bin[row_bin(EMPTY32)], parts);
        lds_add(&bin[NSGC_GRID_MAX_SUB + col_bin(EMPTY32)], parts);
      }
    }
    if (round == 0) {
      special = misc[1];
      starts();
      if (failed)   // slots left over hold empty entries (no packets), which phase C skips
        for (uint32_t i = tid; i < total; i += NT) {
          er[i] = 0ull;
          ec[i] = 0ull;
        }
    }
    __syncthreads();   // (the empty entries land before any emission)
    auto emit = [&](u64 k, uint32_t n) {
      const uint32_t r = uint32_t(k >> 32), c = uint32_t(k);
      ++links;
      mx = max(mx, n);
      emit_row(r, n);
      emit_col(c, n);
      if (!row_light(r)) add_heavy(0, r, n);
      if (!col_light(c)) add_heavy(1, c, n);
    };
    for (uint32_t s = tid; s < SL; s += NT)
      if (tk[s] != EMPTY64) emit(tk[s], tc[s]);
    if (tid == 0 && special && round == 0) emit(EMPTY64, special);
    if (fill[2] == 0) break;
  }
  __syncthreads();
  if (abandoned) {   // empty segments, so that phase C reads nothing here
    for (uint32_t i = tid; i < rsub + csub + 3; i += NT) rec[i] = 0;
  }
  if (tid < 4) misc[tid] = 0;
  __syncthreads();
  links = wave_sum(links);
  mx = wave_max(mx);
  if (lane == 0) {
    lds_add(&misc[2], links);
    __hip_atomic_fetch_max(&misc[3], mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
  if (tid < 2 * HV) gptr(W.acc)[u64(cell) * (2 * HV) + tid] = acc[tid];
  if (tid == 0) {
    const v4u32 part = {total, misc[2], misc[3], abandoned ? 1u : 0u};
    gptr(reinterpret_cast<v4u32*>(W.partB))[cell] = part;
  }
  __syncthreads();
  }
}

// The phase in three sizes: SMALL and BIG for windows of smaller and of larger
// cells, and WIDE for the cells that the others listed as too large for them and
// for windows whose cells have more packets on average than BIG's threads hold,
// with three times the keys and twice the table (one workgroup per compute unit).
// Cells that SMALL or WIDE list go to k_grid_rounds.  Sixteen windows of 2^23
// packets among 4096 addresses, half of whose cells overflow BIG, took 8.2 ms
// without WIDE and take 3.7 ms with it.
enum GridCells { SMALL, BIG, WIDE };

template <int NT, int SL, int E, GridCells KIND>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(KIND == WIDE ? 4 : 6))) void k_grid_links(
    nsgc_dev_plan* P) {
  constexpr int NW = NT / 64;
  constexpr uint32_t ROOM = NT * E;
  static_assert(ROOM * 4 <= SL * 8, "the positions share the key table");
  static_assert((2 * NT + 2 * NW) * 4 <= SL * 2, "the segment table shares the counts");
  static_assert(ROOM < 65536, "16-bit counts");
  static_assert(KIND != BIG || (ROOM == NSGC_GRID_BIG_KEYS && NT == NSGC_GRID_BIG_TILES), "see the planner's classes");
  static_assert(KIND != SMALL || NT == NSGC_GRID_SMALL_TILES, "see the planner's classes");
  __shared__ __align__(16) u64 tk[SL];
  __shared__ __align__(16) uint32_t tc[SL / 2];   // 16-bit counts, two to a word
  __shared__ u64 acc[2 * HVM];
  __shared__ uint32_t bin[2 * NSGC_GRID_MAX_SUB];   // rows, columns
  __shared__ uint32_t misc[8];   // 0 failed, 1 special packets, 2 links, 3 max packets, 7 queue slot
  const uint32_t lane = lane_id();
  // WIDE: the cells of its own windows, then the listed ones
  const uint32_t own = KIND == WIDE  ? sload(&P->gitemsB) - sload(&P->gitemsW)
                       : KIND == BIG ? sload(&P->gitemsW) - sload(&P->gitemsS)
                                     : sload(&P->gitemsS);
  const uint32_t items = own + (KIND == WIDE ? gptr(&P->gover[0])[0] : 0u);
  auto item_at = [&](uint32_t pos) -> uint32_t {
    if (KIND == WIDE && pos >= own) return uniform(gptr(sload(&P->goverB))[pos - own]);
    return uniform((KIND == WIDE ? sload(&P->gitemsW) : KIND == BIG ? sload(&P->gitemsS) : 0u) + pos);
  };
  const uint32_t T = 1u << sload(&P->gtile_log2);

  const uint32_t HV = NSGC_GRID_HV(sload(&P->gtile_log2));
  if (threadIdx.x < 2 * HV) acc[threadIdx.x] = 0;

  GridQueue q(gptr(&sload(&P->queue)[NSGC_Q_GRID + KIND][0]), items);
  // This thread's tile record of item `it` (lane or thread t: tile t), loaded
  // for the next item while the current one is worked on.
  auto record = [&](const nsgc_grid_desc& W, uint32_t it, uint32_t t) -> uint32_t {
    if (W.ntiles <= 64) t &= 63u;
    const uint32_t cells = 1u << (W.subA + W.subB);
    return t < W.ntiles ? gptr(W.tile)[u64(t) * cells + (it - W.itemB)] : 0u;
  };
  uint32_t x = 0, wnext = 0;   // the next item's record and window
  bool have = false;
  for (uint32_t pos0 = blockIdx.x < items ? blockIdx.x : NO_ITEM; pos0 != NO_ITEM;) {
    // opaque, so that what depends on it is computed per item and does not
    // hold registers across items
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const uint32_t it = item_at(pos0);
    if (!have) wnext = sload(sload(&P->gitemB) + it);
    const nsgc_grid_desc W = sload_words(sload(&P->gwin) + wnext);
    const uint32_t cell = it - W.itemB, wcur = wnext;
    const uint32_t nt = W.ntiles;

    // the cell's segments (one per tile) and its packets; `below`: the
    // window's keys in cells below this one, the emission base
    uint32_t below = 0, total = ROOM + 1;
    if (!have) {
      x = record(W, it, tid);
      arrived(x);
    }
    q.announce(&misc[6], items);
    below = x & 0xFFFFu;
    if (nt <= 64)
      total = spread_by_wave<NT>(tid, nt, lane * T + (x & 0xFFFFu), x >> 16, below,
                                 reinterpret_cast<uint32_t*>(tk), ROOM);
    else if (KIND == WIDE) {   // a thread per tile, in turns where there are more
      total = 0;
      for (uint32_t t = 0; t < nt && total <= ROOM; t += NT) {
        if (t) {
          lds_barrier();   // the last turn's scratch has been read
          x = record(W, it, t + tid);
        }
        uint32_t more = x & 0xFFFFu;
        total += spread_segments<NT>(tid, min(nt - t, uint32_t(NT)), (t + tid) * T + (x & 0xFFFFu), x >> 16, more,
                                     tc, reinterpret_cast<uint32_t*>(tk) + total, ROOM - total);
        below = t ? below + more : more;
      }
    } else if (nt <= NT) {   // (an outer cell of a large window may have more: left to WIDE)
      total = spread_segments<NT>(tid, nt, tid * T + (x & 0xFFFFu), x >> 16, below, tc,
                                  reinterpret_cast<uint32_t*>(tk), ROOM);
    }
    lds_barrier();
    const uint32_t ahead = uniform(misc[6]);
    have = ahead != NO_ITEM;
    const uint32_t itnext = have ? item_at(ahead) : it;
    wnext = sload(sload(&P->gitemB) + itnext);
    bool done = false;
    uint32_t links = 0, mx = 0;
    if (total <= ROOM) {
      auto home = [&](u64 k) { return link_home(k) & uint32_t(SL - 1); };
      NSGC_GLOBAL u64* keys = gptr(W.keys);
      // only the last cell can hold the key that equals the table's marker
      const bool marker = ((W.strip_i + (cell >> W.subB) + 1u) >> W.logA) != 0 &&
                          ((W.strip_j + (cell & ((1u << W.subB) - 1u)) + 1u) >> W.logBc) != 0;
      const uint32_t kmax = uniform((total + NT - 1) / NT);
      const uint32_t* list = reinterpret_cast<const uint32_t*>(tk);
      const uint16_t* tc16 = reinterpret_cast<const uint16_t*>(tc);
      u64 key[E];
#pragma unroll
      for (int k = 0; k < E; ++k) {
        key[k] = 0;
        if (uint32_t(k) < kmax) {
          const uint32_t e = k * NT + tid;
          key[k] = keys[e < total ? list[e] : 0u];
        }
      }
      lds_barrier();
      clear_cell_table<NT, SL, SL / 2>(tid, tk, tc, bin, misc);
      lds_barrier();
      loads_arrived();
      if (have) x = record(sload_words(sload(&P->gwin) + wnext), itnext, tid);
      uint32_t at[E];   // slot of a link that this thread inserted
#pragma unroll
      for (int k0 = 0; k0 < E; k0 += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) at[k0 + u] = NO_SLOT;
        if (uint32_t(k0) < kmax) {
          // the home slots of four keys together, then each key's probing
          u64 old[4];
          uint32_t s[4];
          bool ok[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            ok[u] = uint32_t((k0 + u) * NT) + tid < total;
            s[u] = home(key[k0 + u]);
            old[u] = key[k0 + u];
          }
          if (marker) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (ok[u] && key[k0 + u] == EMPTY64) {   // counted outside the table
                lds_add(&misc[1], 1);
                ok[u] = false;
              }
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (ok[u]) old[u] = lds_cas64(&tk[s[u]], EMPTY64, key[k0 + u]);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (ok[u]) {
              const u64 o = probe_on<u64>(tk, uint32_t(SL - 1), key[k0 + u], old[u], s[u]);
              if (o == EMPTY64) at[k0 + u] = s[u];
              else if (o == key[k0 + u]) lds_add(&tc[s[u] >> 1], 1u << ((s[u] & 1u) << 4));
              else misc[0] = 1;
            }
          }
        }
      }
      // the next item's record and the queue's answer, before any store
      arrived(x);
      arrived(q.pending);
      lds_barrier();
      done = misc[0] == 0;
      if (done) {
        // (the descriptor again: scalar registers are short above)
        uint32_t wi = wcur;
        asm volatile("" : "+s"(wi));
        const nsgc_grid_desc G = sload_words(sload(&P->gwin) + wi);
        const uint32_t a = G.logA, b = G.logBc;
        const uint32_t ci = G.strip_i + (cell >> G.subB), cj = G.strip_j + (cell & ((1u << G.subB) - 1u));
        const uint32_t rsub = 1u << (G.logR - a), csub = 1u << (G.logC - b);
        NSGC_GLOBAL uint32_t* rec = gptr(G.rec) + u64(cell) * (rsub + csub + 3);
        NSGC_GLOBAL u64* er = gptr(G.emit_row) + G.base + below;
        NSGC_GLOBAL u64* ec = gptr(G.emit_col) + G.base + below;
        auto row_bin = [&](uint32_t r) { return (r >> (32 - G.logR)) & (rsub - 1u); };
        auto col_bin = [&](uint32_t c) { return (c >> (32 - G.logC)) & (csub - 1u); };
        auto row_light = [&](uint32_t r) { return (r >> (32 - a)) == ci; };
        auto col_light = [&](uint32_t c) { return (c >> (32 - b)) == cj; };
        // a link of the dominant source (v = 0) or destination (v = 1) that `id` names
        auto add_heavy = [&](uint32_t v, uint32_t id, uint32_t n) {
          lds_add64(&acc[v * HV + (id & (HV - 1))], (u64(1) << 32) | n);
        };
        const uint32_t special = marker ? misc[1] : 0u;
        uint32_t nf = 0, nr = 0, nc = 0;   // the wavefront's links, and their light entries
        uint32_t rk[E];   // ranks in the row bin | column bin << 16 (several bins)
#pragma unroll
        for (int k = 0; k < E; ++k)   // from here on `at` is the link's packets, 0 for none
          if (uint32_t(k) < kmax) at[k] = at[k] != NO_SLOT ? tc16[at[k]] + 1u : 0u;
#pragma unroll
        for (int k = 0; k < E; ++k) {
          rk[k] = 0;
          if (uint32_t(k) < kmax) {
            const uint32_t r = uint32_t(key[k] >> 32), c = uint32_t(key[k]);
            const bool fr = at[k] != 0, rl = fr && row_light(r), cl = fr && col_light(c);
            nf += __popcll(__ballot(fr));
            mx = max(mx, at[k]);
            if (rsub == 1) nr += __popcll(__ballot(rl));
            else if (rl) rk[k] = lds_add(&bin[row_bin(r)], 1);
            if (csub == 1) nc += __popcll(__ballot(cl));
            else if (cl) rk[k] |= lds_add(&bin[NSGC_GRID_MAX_SUB + col_bin(c)], 1) << 16;
            if (fr && !rl) add_heavy(0, r, at[k]);
            if (fr && !cl) add_heavy(1, c, at[k]);
          }
        }
        uint32_t srk = 0;
        if (tid == 0 && special) {   // its addresses are never dominant
          srk = lds_add(&bin[rsub - 1], 1) | (lds_add(&bin[NSGC_GRID_MAX_SUB + csub - 1], 1) << 16);
          ++nf;
          mx = max(mx, special);
        }
        mx = wave_max(mx);
        uint32_t br = 0, bc = 0;   // single bins: the wavefront's first entry
        if (lane == 0) {
          if (rsub == 1) br = lds_add(&bin[0], nr);
          if (csub == 1) bc = lds_add(&bin[NSGC_GRID_MAX_SUB], nc);
          lds_add(&misc[2], nf);
          __hip_atomic_fetch_max(&misc[3], mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        br = uniform(br);
        bc = uniform(bc);
        lds_barrier();
        uint32_t xr, xc;
        publish_starts(rec, bin, rsub, csub, G.base + below, xr, xc);
#pragma unroll
        for (int k = 0; k < E; ++k) {
          if (uint32_t(k) < kmax) {
            arrived(key[k]);   // (recomputed from the key: registers are short)
            const uint32_t r = uint32_t(key[k] >> 32), c = uint32_t(key[k]);
            const bool rl = at[k] && row_light(r), cl = at[k] && col_light(c);
            uint32_t pr, pc;
            if (rsub == 1) {
              const u64 m = __ballot(rl);
              pr = br + rank_below(m);
              br += __popcll(m);
            } else {
              pr = lane_take(xr, row_bin(r)) + (rk[k] & 0xFFFFu);
            }
            if (csub == 1) {
              const u64 m = __ballot(cl);
              pc = bc + rank_below(m);
              bc += __popcll(m);
            } else {
              pc = lane_take(xc, col_bin(c)) + (rk[k] >> 16);
            }
            const uint32_t lo = (1u << NSGC_ENT_PACKET_BITS) | at[k];   // below 2^19: one entry
            if (rl) er[pr] = (u64(r) << 32) | lo;
            if (cl) ec[pc] = (u64(c) << 32) | lo;
          }
        }
        if (special) {   // the last bin of each strip
          const uint32_t bs = lane_take(xr, rsub - 1), cs = lane_take(xc, csub - 1);
          if (tid == 0) {
            const u64 e = (u64(EMPTY32) << 32) | (u64(1) << NSGC_ENT_PACKET_BITS) | special;
            er[bs + (srk & 0xFFFFu)] = e;
            ec[cs + (srk >> 16)] = e;
          }
        }
        links = misc[2];
        mx = misc[3];
      }
    }
    if (done) {   // (the last write of `acc` is behind a barrier)
      if (tid < 2 * HV) {
        gptr(W.acc)[u64(cell) * (2 * HV) + tid] = acc[tid];
        acc[tid] = 0;
      }
      if (tid == 0) {
        const v4u32 part = {total, links, mx, 0u};
        gptr(reinterpret_cast<v4u32*>(W.partB))[cell] = part;
      }
    } else if (tid == 0) {   // listed for WIDE or k_grid_rounds
      const uint32_t at = __hip_atomic_fetch_add(gptr(&P->gover[KIND == WIDE ? 2 : 0]), 1u, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
      gptr(KIND == WIDE ? sload(&P->goverW) : sload(&P->goverB))[at] = it;
    }
    if (total > ROOM && have) {
      x = record(sload_words(sload(&P->gwin) + wnext), itnext, tid);
      arrived(x);
    }
    pos0 = ahead;
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// Phase C: the sources of one row bucket (or the destinations of one column
// bucket, or a few neighbouring buckets).  A few more items per window add up
// its dominant addresses.  Like phase B one pass over keys in registers, bound
// by the same chain: 64 windows of 2^17 packets in 62 us against 81 us with one
// segment per link bucket.
// ---------------------------------------------------------------------------

constexpr int GC_NT = 512;
constexpr int GC_E = 12;

size_t lds_grid_rc_bytes(uint32_t slots_log2) {
  const size_t table = (size_t(1) << slots_log2) * 12;
  return std::max(table, size_t(GC_NT) * GC_E * 4) + (2 * GC_NT + 2 * GC_NT / 64 + 64) * 4;
}

template <int NT>
__device__ __forceinline__ void clear_id_table(uint32_t tid, u64* tv, uint32_t* tk, uint32_t S, uint32_t* misc) {
  const v4u32 e4 = {EMPTY32, EMPTY32, EMPTY32, EMPTY32}, z4 = {0u, 0u, 0u, 0u};
  for (uint32_t i = tid; i < S / 2; i += NT) reinterpret_cast<v4u32*>(tv)[i] = z4;
  for (uint32_t i = tid; i < S / 4; i += NT) reinterpret_cast<v4u32*>(tk)[i] = e4;
  if (tid < 4) misc[tid] = 0;
}

// What phase-C item k of a window is: one of the items of the dominant
// addresses (`heavy`: 1 sources, 2 destinations, a few of them from slot `sub`;
// 3 the links between them; first in the window, since they are chains of
// loads), row buckets, or column buckets (1 << group of them, neighbours in one
// strip).
struct BucketItem {
  uint32_t heavy, row, last, group, strip, sub, nseg, word;
};
__device__ __forceinline__ BucketItem bucket_item(const nsgc_grid_desc& W, uint32_t HV, uint32_t k) {
  BucketItem B;
  const uint32_t R = 1u << W.logRi, H = NSGC_GRID_CITEMS(HV) - 1u;
  B.heavy = k > H ? 0u : k == H ? 3u : 1u + k / (H / 2u);
  const uint32_t of_view = k % (H / 2u);
  k -= B.heavy ? 0u : H + 1u;
  B.row = k < R;
  if (!B.row) k -= R;
  const uint32_t items = B.row ? W.logRi : W.logCi, strips = B.row ? W.logA : W.logBc;
  B.last = k + 1u == (1u << items);
  B.group = (B.row ? W.logR : W.logC) - items;
  B.strip = k >> (items - strips);
  B.sub = (k << B.group) & ((1u << (items - strips + B.group)) - 1u);
  if (B.heavy) B.sub = of_view << NSGC_GRID_HV_ITEM_LOG2(HV);
  B.nseg = B.row ? 1u << W.logBc : 1u << W.logA;   // cells of the strip
  B.word = (B.row ? 1u : 2u + (1u << (W.logR - W.logA))) + B.sub;   // its first start in a cell record
  return B;
}
// Word offset of the record of cell s of the item's strip.
__device__ __forceinline__ u64 bucket_record(const nsgc_grid_desc& W, const BucketItem& B, uint32_t s) {
  const uint32_t i = B.row ? B.strip : s, j = B.row ? s : B.strip;
  const uint32_t sub = ((i & ((1u << W.subA) - 1u)) << W.subB) | (j & ((1u << W.subB) - 1u));
  const uint32_t cell = ((((i >> W.subA) << (W.logBc - W.subB)) | (j >> W.subB)) << (W.subA + W.subB)) | sub;
  return u64(cell) * ((1u << (W.logR - W.logA)) + (1u << (W.logC - W.logBc)) + 3u);
}

// The buckets that phase C's single pass listed as too large for it: in a table
// twice as large, one workgroup of 1024 threads per compute unit, and beyond that
// by sweeps over their ids by the bits that follow the bucket's.  Where every
// address is met once all buckets come here: those of 64 windows of 2^17 packets
// in 0.27 ms, against 0.7 ms by sweeps with k_grid_rowcol's table.
constexpr int GS_NT = 1024;
__host__ __device__ constexpr uint32_t sweep_slots_log2(uint32_t slots_log2) {
  return slots_log2 < 12 ? slots_log2 + 1 : 13u;
}

size_t lds_grid_sweep_bytes(uint32_t slots_log2) {
  return (size_t(12) << sweep_slots_log2(slots_log2)) + (3 * (GS_NT / 64) + 16) * 4;
}

__global__ __launch_bounds__(GS_NT) void k_grid_sweeps(nsgc_dev_plan* P) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NT = GS_NT, NW = NT / 64;
  const uint32_t S = 1u << sweep_slots_log2(sload(&P->rc_slots_log2));
  u64* tv = reinterpret_cast<u64*>(smem);
  uint32_t* tk = reinterpret_cast<uint32_t*>(tv + S);
  uint32_t* red = tk + S;    // [3 * NW]
  uint32_t* misc = red + 3 * NW;
  const uint32_t tid = threadIdx.x;
  const uint32_t items = P->gover[1], HV = NSGC_GRID_HV(sload(&P->gtile_log2));
  for (uint32_t x = blockIdx.x; x < items; x += gridDim.x) {
  const uint32_t it = uniform(gptr(sload(&P->goverC))[2 * u64(x)]);
  const uint32_t lo = uniform(gptr(sload(&P->goverC))[2 * u64(x) + 1]);
  const nsgc_grid_desc W = sload_words(sload(&P->gwin) + sload(sload(&P->gitemC) + it));
  const BucketItem B = bucket_item(W, HV, it - W.itemC);
  const uint32_t nseg = B.nseg, logK = B.row ? W.logR : W.logC;
  const NSGC_GLOBAL uint32_t* rec = gptr(W.rec);
  const NSGC_GLOBAL u64* em = gptr(B.row ? W.emit_row : W.emit_col);
  auto seg = [&](uint32_t s, u64& base, uint32_t& len) {
    const NSGC_GLOBAL uint32_t* x = rec + bucket_record(W, B, s);
    const uint32_t s0 = x[B.word + lo], s1 = x[B.word + lo + 1];
    base = u64(x[0]) + s0;
    len = s1 - s0;
  };
  uint32_t n = 0, mp = 0, ml = 0;
  bool abandoned = false;
  // sweeps over the bucket's ids by the bits that follow the bucket's
  for (uint32_t logS = 0;; ++logS) {
    if (logS > sload(&P->max_sweeps_log2)) { abandoned = true; break; }
    n = mp = ml = 0;
    bool failed = false;
    for (uint32_t sw = 0; sw < (1u << logS) && !failed; ++sw) {
      __syncthreads();
      clear_id_table<NT>(tid, tv, tk, S, misc);
      __syncthreads();
      gather_by_wave<4, NW>(nseg, seg, [&](const auto& pos, const auto& okin) {
        constexpr int U = array_len<decltype(pos)>();
        uint32_t id[U], pk[U], ln[U], at[U];
        bool ok[U], fr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const u64 x = em[okin[u] ? pos[u] : 0ull];
          id[u] = uint32_t(x >> 32);
          pk[u] = uint32_t(x) & ENT_PMAX;
          ln[u] = uint32_t(x) >> NSGC_ENT_PACKET_BITS;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          at[u] = id[u] & (S - 1);
          ok[u] = okin[u] && pk[u] != 0 && !(logS && next32(id[u], logK, logS) != sw);
          if (ok[u] && id[u] == EMPTY32) {
            lds_add(&misc[2], pk[u]);
            lds_add(&misc[3], ln[u]);
            ok[u] = false;
          }
          // combine the lanes holding the first valid lane's id
          const u64 vm = __ballot(ok[u]);
          if (vm) {
            const int f = __ffsll(static_cast<unsigned long long>(vm)) - 1;
            const bool same = ok[u] && id[u] == readlane(id[u], f);
            if (__popcll(__ballot(same)) > 1) {
              const uint32_t tot = wave_sum(same ? pk[u] : 0u);
              const uint32_t lns = wave_sum(same ? ln[u] : 0u);
              if (same) {
                if (int(lane_id()) == f) { pk[u] = tot; ln[u] = lns; }
                else ok[u] = false;
              }
            }
          }
        }
        if (insert_keys<U>(tk, S - 1, id, at, ok, fr)) lds_store(&misc[0], 1);
#pragma unroll
        for (int u = 0; u < U; ++u)   // (a sweep that failed is thrown away)
          if (ok[u]) lds_add64(&tv[at[u]], (u64(ln[u]) << 32) | pk[u]);
      });
      failed = misc[0] != 0;
      if (!failed) {
        for (uint32_t i = tid; i < S; i += NT)
          if (tk[i] != EMPTY32) {
            ++n;
            mp = max(mp, uint32_t(tv[i]));
            ml = max(ml, uint32_t(tv[i] >> 32));
          }
        if (tid == 0 && misc[3]) {
          ++n;
          mp = max(mp, misc[2]);
          ml = max(ml, misc[3]);
        }
      }
    }
    if (!failed) break;
  }
  __syncthreads();
  block_sum_max2_to0<NW>(n, mp, ml, red);
  if (tid == 0) {   // onto what the single passes found in the item's other buckets
    NSGC_GLOBAL uint32_t* o = gptr(W.partC) + u64(it - W.itemC) * 4;
    __hip_atomic_fetch_add(o, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(o + 1, mp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(o + 2, ml, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(o + 3, abandoned ? 1u : 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  }
}

__global__ __launch_bounds__(GC_NT) __attribute__((amdgpu_waves_per_eu(6))) void k_grid_rowcol(
    nsgc_dev_plan* P) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NT = GC_NT, E = GC_E, NW = NT / 64;
  constexpr uint32_t ROOM = NT * E;
  const uint32_t S = 1u << sload(&P->rc_slots_log2);
  // [S] links << 32 | packets, [S] ids; the element positions share them
  u64* tv = reinterpret_cast<u64*>(smem);
  uint32_t* tk = reinterpret_cast<uint32_t*>(tv + S);
  uint32_t* list = reinterpret_cast<uint32_t*>(smem);
  uint32_t* tab = reinterpret_cast<uint32_t*>(smem + max(S * 12u, ROOM * 4u));
  uint32_t* red = tab + 2 * NT + 2 * NW;   // [3 * NW]
  uint32_t* misc = red + 32;               // 0 failed, 2 / 3 marker id's packets / links, 7 queue slot
  const uint32_t items = sload(&P->gitemsC), HV = NSGC_GRID_HV(sload(&P->gtile_log2));

  GridQueue q(gptr(&sload(&P->queue)[NSGC_Q_GRID_C][0]), items);
  // This thread's segment of buckets lo .. lo + w - 1 (all, if w is 0) of item
  // `it`, cell `s` of its strip: emission base and length.  The next item's is
  // loaded while the current one is worked on.
  struct Segment { uint32_t cell, start, end; };   // the cell's base, starts relative to it
  auto segment = [&](uint32_t it, uint32_t lo, uint32_t w, uint32_t s) -> Segment {
    const nsgc_grid_desc W = sload_words(sload(&P->gwin) + sload(sload(&P->gitemC) + it));
    const BucketItem B = bucket_item(W, HV, it - W.itemC);
    Segment g = {0, 0, 0};
    if (B.heavy) return g;
    if (w == 0) w = 1u << B.group;
    if (B.nseg <= 64) s &= 63u;
    if (s >= B.nseg) return g;
    const NSGC_GLOBAL uint32_t* x = gptr(W.rec) + bucket_record(W, B, s);
    const NSGC_GLOBAL uint32_t* y = x + B.word + lo;
    g.cell = x[0];
    g.start = y[0];
    g.end = y[w];
    return g;
  };
  Segment sg = {0, 0, 0};
  bool have = false;
  for (uint32_t item = blockIdx.x < items ? blockIdx.x : NO_ITEM; item != NO_ITEM;) {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // (as in phase B)
    const uint32_t it = uniform(item);
    const nsgc_grid_desc W = sload_words(sload(&P->gwin) + sload(sload(&P->gitemC) + it));
    const BucketItem B = bucket_item(W, HV, it - W.itemC);
    uint32_t n = 0, mp = 0, ml = 0;
    if (!have) {
      sg = segment(it, 0, 0, tid);
      loads_arrived();
    }
    q.announce(misc + 6, items);
    Segment ng = {0, 0, 0};
    uint32_t ahead = NO_ITEM;
    bool loaded = false;
    auto look_ahead = [&]() {   // (a barrier has passed since the next item was announced)
      ahead = uniform(misc[6]);
      have = ahead != NO_ITEM;
      if (have) ng = segment(ahead, 0, 0, tid);
      loaded = true;
    };
    if (B.heavy) {
      const uint32_t k = B.heavy - 1u;
      const NSGC_GLOBAL uint32_t* m = gptr(W.heavy) + 2 * HV;
      if (k == 2) {   // links between dominant addresses: packets, links, maximum
        for (uint32_t i = tid; i < HV * HV; i += NT) {
          const uint32_t x = m[i];
          n += x;
          mp += x ? 1u : 0u;
          ml = max(ml, x);
        }
        block_sum2_max_to0<NW>(n, mp, ml, red);
      } else {        // dominant sources (destinations): the cells' counters and the matrix
        const uint32_t G = 1u << NSGC_GRID_HV_ITEM_LOG2(HV), stride = NT >> NSGC_GRID_HV_ITEM_LOG2(HV);
        u64* sum = tv;
        const uint32_t s = B.sub + (tid & (G - 1u)), g = tid >> NSGC_GRID_HV_ITEM_LOG2(HV);
        const uint32_t cells = 1u << W.logP;
        const NSGC_GLOBAL u64* acc = gptr(W.acc) + k * HV + s;
        u64 x = 0;
#pragma unroll 16
        for (uint32_t cell = g; cell < cells; cell += stride) x += acc[u64(cell) * (2 * HV)];
        for (uint32_t o = g; o < HV; o += stride) {
          const uint32_t y = k == 0 ? m[s * HV + o] : m[o * HV + s];
          x += (u64(y ? 1u : 0u) << 32) | y;
        }
        sum[tid] = x;
        lds_barrier();
        if (tid < 64) {
          for (uint32_t o = 1; o < NW; ++o) x += sum[o * 64 + tid];
          for (uint32_t o = G; o < 64; o *= 2) x += __shfl_xor(x, int(o));
          if (tid < G) {
            n = (x >> 32) ? 1u : 0u;
            mp = uint32_t(x);
            ml = uint32_t(x >> 32);
          }
        }
        block_sum_max2_to0<NW>(n, mp, ml, red);
      }
    } else {
      const NSGC_GLOBAL u64* em = gptr(B.row ? W.emit_row : W.emit_col);
      // the item's buckets in one pass if they fit it, else in halves, quarters, ...
      uint32_t w = 1u << B.group;
      bool reload = false;
      for (uint32_t lo = 0; lo < (1u << B.group);) {
      if (reload) {
        sg = segment(it, lo, w, tid);
        loads_arrived();
      }
      reload = true;
      uint32_t none = 0;
      const uint32_t total =
          B.nseg <= 64
              ? spread_by_wave<NT>(tid, B.nseg, sg.cell + sg.start, sg.end - sg.start, none, list, ROOM)
              : spread_segments<NT>(tid, B.nseg, sg.cell + sg.start, sg.end - sg.start, none, tab, list, ROOM);
      lds_barrier();
      bool done = false;
      // the last bucket holds the id that equals the tables' marker
      const bool last = B.last && lo + w == (1u << B.group);
      if (total <= ROOM) {
        const uint32_t kmax = uniform((total + NT - 1) / NT);
        u64 e[E];
#pragma unroll
        for (int j = 0; j < E; ++j) {
          e[j] = 0;
          if (uint32_t(j) < kmax) {
            const uint32_t x = uint32_t(j * NT) + tid;
            e[j] = em[x < total ? list[x] : 0u];   // masked when it is used
          }
        }
        lds_barrier();
        clear_id_table<NT>(tid, tv, tk, S, misc);
        lds_barrier();
        loads_arrived();
        if (!loaded) look_ahead();
        uint32_t at[E];   // slot of an id that this thread inserted
#pragma unroll
        for (int j0 = 0; j0 < E; j0 += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) at[j0 + u] = NO_SLOT;
          if (uint32_t(j0) < kmax && !lds_load(&misc[0])) {   // (a pass that failed is thrown away)
            uint32_t id[4], lo[4], old[4], s[4];
            bool ok[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              id[u] = uint32_t(e[j0 + u] >> 32);
              lo[u] = uint32_t(e[j0 + u]);
              // (an entry with no packets is an unused slot of a cell that took rounds)
              ok[u] = uint32_t((j0 + u) * NT) + tid < total && (lo[u] & ENT_PMAX) != 0;
              s[u] = id[u] & (S - 1);
              old[u] = id[u];
            }
            if (last) {
#pragma unroll
              for (int u = 0; u < 4; ++u)
                if (ok[u] && id[u] == EMPTY32) {
                  lds_add(&misc[2], lo[u] & ENT_PMAX);
                  lds_add(&misc[3], lo[u] >> NSGC_ENT_PACKET_BITS);
                  ok[u] = false;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (ok[u]) old[u] = lds_cas32(&tk[s[u]], EMPTY32, id[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (ok[u]) {
                const uint32_t o = probe_on<uint32_t>(tk, S - 1, id[u], old[u], s[u]);
                if (o == EMPTY32) at[j0 + u] = s[u];
                else if (o != id[u]) misc[0] = 1;
                lds_add64(&tv[s[u]], (u64(lo[u] >> NSGC_ENT_PACKET_BITS) << 32) | (lo[u] & ENT_PMAX));
              }
            }
            // entries for more than 15/16 of the table and hardly an id met twice yet:
            // it will overflow
            if (j0 == 0 && total > S - S / 16) {
              uint32_t fresh = 0;
#pragma unroll
              for (int u = 0; u < 4; ++u) fresh += __popcll(__ballot(at[u] != NO_SLOT));
              if (fresh > 4 * 64 - 4) misc[0] = 1;
            }
          }
        }
        lds_barrier();
        if (misc[0] == 0) {
          done = true;
#pragma unroll
          for (int j = 0; j < E; ++j)
            if (at[j] != NO_SLOT) {
              const u64 x = tv[at[j]];
              ++n;
              mp = max(mp, uint32_t(x));
              ml = max(ml, uint32_t(x >> 32));
            }
          if (tid == 0 && misc[3]) {
            ++n;
            mp = max(mp, misc[2]);
            ml = max(ml, misc[3]);
          }
        }
      }
      lds_barrier();   // the table is free again
      if (!done && w > 1) {
        w >>= 1;
        continue;
      }
      if (!done && tid == 0) {   // a single bucket, left to k_grid_sweeps
        const uint32_t at = __hip_atomic_fetch_add(gptr(&P->gover[1]), 1u, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
        gptr(sload(&P->goverC))[2 * u64(at)] = it;
        gptr(sload(&P->goverC))[2 * u64(at) + 1] = lo;
      }
      lo += w;
      }
      block_sum_max2_to0<NW>(n, mp, ml, red);
    }
    if (!loaded) look_ahead();
    // the next item's segment and the queue's answer, before the store
    loads_arrived();
    arrived(q.pending);
    if (tid == 0) {
      const v4u32 part = {n, mp, ml, 0u};
      gptr(reinterpret_cast<v4u32*>(W.partC))[it - W.itemC] = part;
    }
    sg = ng;
    item = ahead;
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// Phase C for the entity counts (nsgc_window_entity_counts): destinations are
// hashed like sources and both views have the same buckets, so item k takes row
// bucket k and column bucket k into one table of ids with a mark per view; its
// marked slots are the item's share of sources, destinations and their union.
// The bucket's dominant addresses, which emit no entries, are put in by hand.
// In sweeps over the ids, streaming the entries, where a bucket has more
// entries than the threads hold or more ids than the table.  Bound by its chain
// like k_grid_rowcol; nothing but marks is kept, so the table costs 49 KB.
// Counts of 64 windows of 2^17 packets 48 us (300 by k_rowcol_ent, whose item
// reads one segment per link bucket), whole calls 451 -> 179 us; one window of
// 2000 packets 46 -> 31, so every window above small_max takes the grid.
// ---------------------------------------------------------------------------

constexpr int GE_NT = 512;
constexpr int GE_E = 8;
constexpr uint32_t GE_S = 8192;

__global__ __launch_bounds__(GE_NT) __attribute__((amdgpu_waves_per_eu(6))) void k_grid_ent(nsgc_dev_plan* P) {
  constexpr int NT = GE_NT, E = GE_E, NW = NT / 64;
  constexpr uint32_t S = GE_S, ROOM = NT * E;
  __shared__ __align__(16) uint32_t tk[S];        // ids; before them the positions of a view's entries
  __shared__ __align__(16) uint8_t mark[2][S];
  __shared__ uint32_t tab[2 * NT + 2 * NW];
  __shared__ uint32_t misc[8];   // 0 failed, 1 / 2 the tables' marker seen as source / destination, 6 next item
  __shared__ uint32_t red[3 * NW];
  static_assert(S / 16 == NT, "a thread per 16 slots");
  const uint32_t items = sload(&P->gitemsC), HV = NSGC_GRID_HV(sload(&P->gtile_log2));
  GridQueue q(gptr(&sload(&P->queue)[NSGC_Q_GRID_C][0]), items);
  for (uint32_t item = blockIdx.x < items ? blockIdx.x : NO_ITEM; item != NO_ITEM;) {
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // (as in phase B)
    const uint32_t it = uniform(item);
    const nsgc_grid_desc W = sload_words(sload(&P->gwin) + sload(sload(&P->gitemC) + it));
    const uint32_t k = it - W.itemC, H = NSGC_GRID_CITEMS(HV);
    q.announce(misc + 6, items);
    v4u32 part = {0u, 0u, 0u, 0u};
    if (k < H) {
      if (k == H - 1) {   // links between dominant addresses: packets, links, maximum
        const NSGC_GLOBAL uint32_t* m = gptr(W.heavy) + 2 * HV;
        uint32_t n = 0, l = 0, mx = 0;
        for (uint32_t i = tid; i < HV * HV; i += NT) {
          const uint32_t x = m[i];
          n += x;
          l += x ? 1u : 0u;
          mx = max(mx, x);
        }
        block_sum2_max_to0<NW>(n, l, mx, red);
        part.x = n;
        part.y = l;
        part.z = mx;
      }
    } else {
      const uint32_t bucket = k - H, logK = W.logR;
      const bool last = bucket + 1u == (1u << logK);   // holds the id that equals the table's marker
      const NSGC_GLOBAL uint32_t* rec = gptr(W.rec);
      // segment s of the bucket's entries in view v
      auto segment = [&](uint32_t v, uint32_t s, uint32_t& base, uint32_t& len) {
        BucketItem B;
        const uint32_t low = W.logR - (v ? W.logBc : W.logA);
        B.row = v == 0;
        B.strip = bucket >> low;
        B.sub = bucket & ((1u << low) - 1u);
        const NSGC_GLOBAL uint32_t* x = rec + bucket_record(W, B, s);
        const NSGC_GLOBAL uint32_t* y = x + (v ? 2u + (1u << (W.logR - W.logA)) : 1u) + B.sub;
        base = x[0] + y[0];
        len = y[1] - y[0];
      };
      auto insert = [&](uint32_t v, uint32_t id, uint32_t probes) {
        if (last && id == EMPTY32) {
          misc[1 + v] = 1;
          return;
        }
        uint32_t s = id & (S - 1);
        const uint32_t o = probe_on<uint32_t>(tk, S - 1, id, lds_cas32(&tk[s], EMPTY32, id), s, probes);
        if (o == EMPTY32 || o == id) mark[v][s] = 1;
        else misc[0] = 1;
      };
      auto clear = [&]() {
        const v4u32 e4 = {EMPTY32, EMPTY32, EMPTY32, EMPTY32}, z4 = {0u, 0u, 0u, 0u};
#pragma unroll
        for (uint32_t i = 0; i < S / 4 / NT; ++i) reinterpret_cast<v4u32*>(tk)[i * NT + tid] = e4;
#pragma unroll
        for (uint32_t i = 0; i < S / 8 / NT; ++i) reinterpret_cast<v4u32*>(&mark[0][0])[i * NT + tid] = z4;
        if (tid < 3) misc[tid] = 0;
      };
      uint32_t nr = 0, nc = 0, uni = 0;
      auto harvest = [&]() {
        const v4u32 a = reinterpret_cast<const v4u32*>(mark[0])[tid], b = reinterpret_cast<const v4u32*>(mark[1])[tid];
        nr += __popc(a.x) + __popc(a.y) + __popc(a.z) + __popc(a.w);
        nc += __popc(b.x) + __popc(b.y) + __popc(b.z) + __popc(b.w);
        uni += __popc(a.x | b.x) + __popc(a.y | b.y) + __popc(a.z | b.z) + __popc(a.w | b.w);
        if (tid == 0) {
          nr += misc[1];
          nc += misc[2];
          uni += misc[1] | misc[2];
        }
      };
      // the dominant addresses of the bucket (each occurs in the window), and
      // those of sweep sw of 2^logS
      auto dominant = [&](uint32_t logS, uint32_t sw) {
        if (tid < 2 * HV) {
          const uint32_t id = gptr(W.heavy)[tid];
          if (id != EMPTY32 && (id >> (32 - logK)) == bucket && !(logS && next32(id, logK, logS) != sw))
            insert(tid < HV ? 0u : 1u, id, S);
        }
      };
      bool done = false;
      u64 e[2][E];
      uint32_t total[2];
      auto read = [&](uint32_t v) {   // a view's entries into registers
        const uint32_t nseg = 1u << (v ? W.logA : W.logBc);
        const uint32_t s = nseg <= 64 ? tid & 63u : tid;
        uint32_t base = 0, len = 0, none = 0;
        if (s < nseg) segment(v, s, base, len);
        lds_barrier();   // the last list has been read
        const uint32_t n = nseg <= 64 ? spread_by_wave<NT>(tid, nseg, base, len, none, tk, ROOM)
                                      : spread_segments<NT>(tid, nseg, base, len, none, tab, tk, ROOM);
        lds_barrier();
        const NSGC_GLOBAL u64* em = gptr(v ? W.emit_col : W.emit_row);
        if (n <= ROOM) {
#pragma unroll
          for (int j = 0; j < E; ++j) {
            const uint32_t x = uint32_t(j * NT) + tid;
            e[v][j] = 0;
            if (uint32_t(j * NT) < n) e[v][j] = em[x < n ? tk[x] : 0u];   // masked when it is used
          }
        }
        total[v] = n;
      };
      read(0);
      read(1);
      if (total[0] <= ROOM && total[1] <= ROOM) {
        lds_barrier();
        clear();
        lds_barrier();
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
          for (int j = 0; j < E; ++j)
            // (an entry with no packets is an unused slot of a cell that took rounds)
            if (uint32_t(j * NT) + tid < total[v] && (uint32_t(e[v][j]) & ENT_PMAX) != 0)
              insert(uint32_t(v), uint32_t(e[v][j] >> 32), NSGC_MAX_PROBES);
        dominant(0, 0);
        lds_barrier();
        done = misc[0] == 0;
        if (done) harvest();
      }
      bool abandoned = false;
      for (uint32_t logS = 0; !done; ++logS) {
        if (logS > sload(&P->max_sweeps_log2)) { abandoned = true; break; }
        nr = nc = uni = 0;
        bool failed = false;
        for (uint32_t sw = 0; sw < (1u << logS) && !failed; ++sw) {
          __syncthreads();
          clear();
          __syncthreads();
          for (uint32_t v = 0; v < 2; ++v) {
            const NSGC_GLOBAL u64* em = gptr(v ? W.emit_col : W.emit_row);
            auto seg = [&](uint32_t s, u64& base, uint32_t& len) {
              uint32_t b;
              segment(v, s, b, len);
              base = b;
            };
            gather_by_wave<4, NW>(1u << (v ? W.logA : W.logBc), seg, [&](const auto& pos, const auto& okin) {
              constexpr int U = array_len<decltype(pos)>();
              u64 x[U];
#pragma unroll
              for (int u = 0; u < U; ++u) x[u] = em[okin[u] ? pos[u] : 0ull];
#pragma unroll
              for (int u = 0; u < U; ++u) {
                const uint32_t id = uint32_t(x[u] >> 32);
                bool ok = okin[u] && (uint32_t(x[u]) & ENT_PMAX) != 0 && !(logS && next32(id, logK, logS) != sw);
                // one of the lanes with the first valid lane's id
                const u64 vm = __ballot(ok);
                if (vm) {
                  const int f = __ffsll(static_cast<unsigned long long>(vm)) - 1;
                  ok = ok && (int(lane_id()) == f || id != readlane(id, f));
                }
                if (ok) insert(v, id, NSGC_MAX_PROBES);
              }
            });
          }
          dominant(logS, sw);
          __syncthreads();
          failed = misc[0] != 0;
          if (!failed) harvest();
        }
        done = !failed;
      }
      uint32_t none = 0, zero = 0;
      block_sum2_max_to0<NW>(nr, nc, none, red);
      lds_barrier();
      block_sum2_max_to0<NW>(uni, zero, none, red);
      part.x = nr;
      part.y = nc;
      part.z = uni;
      part.w = abandoned ? 1u : 0u;
    }
    lds_barrier();
    item = uniform(misc[6]);
    loads_arrived();
    arrived(q.pending);
    if (tid == 0) gptr(reinterpret_cast<v4u32*>(W.partC))[k] = part;
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------

namespace {
typedef void (*part_fn)(const nsgc_dev_plan*, uint32_t);
part_fn partition_kernel(uint32_t tile_log2, int* threads, bool keys = false) {
  *threads = tile_log2 >= 14 ? 1024 : 512;
  switch (tile_log2) {
    case 11: return &k_grid_partition<4, 512, NSGC_GRID_HV(11)>;
    case 12: return &k_grid_partition<8, 512, NSGC_GRID_HV(12)>;
    case 13: return &k_grid_partition<16, 512, NSGC_GRID_HV(13)>;
    case 14:
      return keys ? &k_grid_partition<16, 1024, NSGC_GRID_HV(14), true>
                  : &k_grid_partition<16, 1024, NSGC_GRID_HV(14)>;
    default: return nullptr;
  }
}
constexpr int GB_NT[3] = {256, 512, 1024};
void (*const links_kernels[3])(nsgc_dev_plan*) = {
    &k_grid_links<GB_NT[0], 2048, 8, SMALL>,
    &k_grid_links<GB_NT[1], 4096, 8, BIG>,
    &k_grid_links<GB_NT[2], 8192, 12, WIDE>,
};
}  // namespace

hipError_t launch_grid_heavy(const nsgc_dev_plan* P, uint32_t tile_log2, uint32_t grid, hipStream_t s) {
  if (NSGC_GRID_HV(tile_log2) == 64)
    hipLaunchKernelGGL((k_grid_heavy<64>), dim3(grid), dim3(GH_NT), 0, s, P);
  else
    hipLaunchKernelGGL((k_grid_heavy<32>), dim3(grid), dim3(GH_NT), 0, s, P);
  return hipGetLastError();
}

hipError_t launch_grid_partition(const nsgc_dev_plan* P, uint32_t tile_log2, uint32_t max_cells,
                                 uint32_t grid, hipStream_t s, bool keys) {
  int threads = 0;
  const part_fn f = partition_kernel(tile_log2, &threads, keys);
  if (!f) return hipErrorInvalidValue;
  hipLaunchKernelGGL(f, dim3(grid), dim3(threads), lds_grid_part_bytes(tile_log2, max_cells), s, P,
                     max_cells);
  return hipGetLastError();
}

hipError_t launch_grid_links(const nsgc_dev_plan* P, int which, uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(links_kernels[which], dim3(grid), dim3(GB_NT[which]), 0, s, const_cast<nsgc_dev_plan*>(P));
  return hipGetLastError();
}

hipError_t launch_grid_rounds(const nsgc_dev_plan* P, bool after_wide, uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(k_grid_rounds, dim3(grid), dim3(GR_NT), 0, s, const_cast<nsgc_dev_plan*>(P),
                     after_wide ? 1u : 0u);
  return hipGetLastError();
}

hipError_t launch_grid_sweeps(const nsgc_dev_plan* P, uint32_t grid, size_t lds, hipStream_t s) {
  hipLaunchKernelGGL(k_grid_sweeps, dim3(grid), dim3(GS_NT), lds, s, const_cast<nsgc_dev_plan*>(P));
  return hipGetLastError();
}

hipError_t launch_grid_rowcol(const nsgc_dev_plan* P, uint32_t grid, size_t lds, hipStream_t s) {
  hipLaunchKernelGGL(k_grid_rowcol, dim3(grid), dim3(GC_NT), lds, s, const_cast<nsgc_dev_plan*>(P));
  return hipGetLastError();
}

hipError_t launch_grid_ent(const nsgc_dev_plan* P, uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(k_grid_ent, dim3(grid), dim3(GE_NT), 0, s, const_cast<nsgc_dev_plan*>(P));
  return hipGetLastError();
}

hipError_t grid_resident_blocks(int which, uint32_t tile_log2, size_t lds, int* blocks) {
  int threads = 0;
  const void* f = nullptr;
  switch (which) {
    case 0: f = reinterpret_cast<const void*>(partition_kernel(tile_log2, &threads)); break;
    case 1: f = reinterpret_cast<const void*>(links_kernels[0]); threads = GB_NT[0]; break;
    case 2: f = reinterpret_cast<const void*>(links_kernels[1]); threads = GB_NT[1]; break;
    case 3: f = reinterpret_cast<const void*>(&k_grid_rowcol); threads = GC_NT; break;
    case 4: f = reinterpret_cast<const void*>(&k_grid_ent); threads = GE_NT; break;
    default: break;
  }
  if (!f) return hipErrorInvalidValue;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, f, threads, lds);
}

hipError_t grid_allow_large_lds(size_t bytes) {
  int t;
  const void* fns[] = {reinterpret_cast<const void*>(partition_kernel(11, &t)),
                       reinterpret_cast<const void*>(partition_kernel(12, &t)),
                       reinterpret_cast<const void*>(partition_kernel(13, &t)),
                       reinterpret_cast<const void*>(partition_kernel(14, &t)),
                       reinterpret_cast<const void*>(partition_kernel(14, &t, true)),
                       reinterpret_cast<const void*>(&k_grid_rowcol),
                       reinterpret_cast<const void*>(&k_grid_sweeps)};
  for (const void* f : fns) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace nsgc
