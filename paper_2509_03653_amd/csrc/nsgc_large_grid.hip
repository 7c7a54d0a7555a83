// Large windows on a grid of two levels: the cells of nsgc_grid.hip, too many
// for one partition tile to hold a run of keys for each, are reached through
// 16 x 16 outer cells.
//
//   1. k_large_count counts the packets of each outer cell in about a thousand
//      ranges of the window, k_large_scan turns the counts into positions, and
//      k_large_split writes every packet's hashed link key into its outer
//      cell's contiguous region (packets between dominant addresses are
//      counted in the matrix instead).
//   2. Every outer cell is a window of its own to k_grid_partition and
//      k_grid_links, with the strips of its part of the grid.
//   3. k_large_reduce adds up the cells' totals and dominant counters per outer
//      cell; k_grid_rowcol sees one window again, whose strips run through the
//      outer cells.
//
// Sorting the keys (nsgc_large.hip) moves 16 bytes per packet in each of eight
// passes and counts them in as many; here a packet's key is written twice and
// read twice.  One skewed window of 3 * 10^8 packets: 30.3 -> 4.4 ms (count
// 0.44, split 1.20, partition 0.60, links 1.73 with the crowded cells, rowcol
// 0.40); 2^24 packets among 4096 addresses 2.20 -> 0.67 ms; 2.9 * 10^8 of the
// benchmark's traffic 40.4 -> 8.1 ms.  Bound by the partition kernels' LDS
// placing (2.4 to 3 TB/s) and by phase B's chain per cell.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "nsgc_device.hpp"
#include "nsgc_grid.hpp"
#include "nsgc_grid_device.hpp"
#include "nsgc_large_grid.hpp"
#include "nsgc_phases.hpp"
#include "nsgc_plan.h"

namespace nsgc {

namespace {

constexpr uint32_t OUT_LOG2 = 4;                     // outer strips, each way
constexpr uint32_t OUT = 1u << (2 * OUT_LOG2);       // outer cells
constexpr uint32_t T = 1u << 14;                     // packets per tile
constexpr uint32_t RANGES = 1024;                    // most ranges of the count
constexpr uint32_t HV = NSGC_GRID_HEAVY;
constexpr uint32_t TILE_LOG2 = 14;
static_assert(NSGC_GRID_HV(TILE_LOG2) == HV, "dominant addresses of 2^14-packet tiles");

// A plan header and its work-queue counters.
constexpr size_t QUEUES = size_t(NSGC_Q_ALL) * NSGC_QCLASSES * NSGC_QSTRIDE * 4;
constexpr size_t HEAD = ((sizeof(nsgc_dev_plan) + 255) / 256 * 256) + QUEUES;

// Where everything lies in the workspace, and the window's grid.
struct Shape {
  uint64_t n;
  uint32_t a, b, logR, logC, logRi, logCi;
  uint32_t cells, items, tiles, per, ranges;   // per: tiles of a range
  size_t keys2, emit_col, tile, rec, heavy, acc, partB, partC, acc2, partB2, goverB, goverW, goverC, itemB,
      itemC, prefA, cnt, win, head, total;
};

int log2_ceil(uint64_t x) {
  int k = 0;
  while ((uint64_t(1) << k) < x) ++k;
  return k;
}

// Cells of 1280 to 2560 packets, up to 2^9 strips each way (a phase-C item
// reads one segment per cell of its strip, one per thread); row and column
// buckets like a grid window's.  From 2^20 packets, the tier's lowest
// threshold, to 2^30, where the cells reach the size of phase B's tables.
bool shape(uint64_t n, Shape* g) {
  if (n < (uint64_t(1) << 20) || n > (uint64_t(1) << 30)) return false;
  const int lc = std::min(std::max(log2_ceil((n + 2559) / 2560), 10), 18);
  g->n = n;
  g->a = uint32_t((lc + 1) / 2);
  g->b = uint32_t(lc / 2);
  const int buckets = log2_ceil((n + NSGC_GRID_BUCKET - 1) / NSGC_GRID_BUCKET);
  g->logR = uint32_t(std::min(std::max(buckets, int(g->a)), int(g->a) + NSGC_GRID_MAX_SUB_LOG2));
  g->logC = uint32_t(std::min(std::max(buckets, int(g->b)), int(g->b) + NSGC_GRID_MAX_SUB_LOG2));
  g->logRi = std::max(g->logR - 2, g->a);
  g->logCi = std::max(g->logC - 2, g->b);
  g->cells = 1u << lc;
  g->items = (1u << g->logRi) + (1u << g->logCi) + NSGC_GRID_CITEMS(HV);
  g->tiles = uint32_t((n + T - 1) / T);
  g->per = (g->tiles + RANGES - 1) / RANGES;
  g->ranges = (g->tiles + g->per - 1) / g->per;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o = (o + bytes + 255) / 256 * 256;
    return at;
  };
  take(size_t(n) * 8);   // the outer cells' keys, then the row entries
  g->keys2 = take(size_t(n) * 8);
  g->emit_col = take(size_t(n) * 8);
  g->tile = take((size_t(n / T) + OUT) * (g->cells / OUT) * 4);
  const size_t sub = (size_t(1) << (g->logR - g->a)) + (size_t(1) << (g->logC - g->b)) + 3;
  g->rec = take(g->cells * sub * 4);
  g->heavy = take(NSGC_GRID_HV_WORDS(HV) * 4);
  g->acc = take(size_t(g->cells) * 2 * HV * 8);
  g->partB = take(size_t(g->cells) * 16);
  g->partC = take(size_t(g->items) * 16);
  g->acc2 = take(size_t(OUT) * 2 * HV * 8);
  g->partB2 = take(size_t(OUT) * 16);
  g->goverB = take(size_t(g->cells) * 4);
  g->goverW = take(size_t(g->cells) * 4);
  g->goverC = take(((size_t(1) << g->logR) + (size_t(1) << g->logC)) * 8);
  g->itemB = take(size_t(g->cells) * 4);
  g->itemC = take(size_t(g->items) * 4);
  g->prefA = take((OUT + 1) * 4);
  g->cnt = take(size_t(g->ranges) * OUT * 4);
  g->win = take((OUT + 1) * sizeof(nsgc_grid_desc));
  g->head = take(2 * HEAD);
  g->total = o;
  return true;
}

// What k_large_init writes down and the other kernels read.
struct Args {
  nsgc_grid_desc W;          // the whole window
  nsgc_grid_desc* win;       // [OUT] the outer cells, then W
  nsgc_dev_plan* inner;      // plan of the outer cells' windows
  nsgc_dev_plan* whole;      // plan of the whole window
  uint32_t* cnt;             // [ranges][OUT]
  uint32_t* prefA;
  uint32_t* itemB;
  uint32_t* itemC;
  uint32_t* goverB;
  uint32_t* goverW;
  uint32_t* goverC;
  unsigned long long* keys2;
  unsigned long long* acc;
  uint32_t* partB;
  unsigned long long* out;
  uint32_t cells, items, per, ranges, rc_slots_log2;
};

// Both plans, the whole window's descriptor, and the windows of the items.
__global__ __launch_bounds__(256) void k_large_init(Args A) {
  const uint32_t tid = blockIdx.x * 256 + threadIdx.x, step = gridDim.x * 256;
  const uint32_t lg = A.W.subA + A.W.subB;
  for (uint32_t i = tid; i < A.cells; i += step) gptr(A.itemB)[i] = i >> lg;
  for (uint32_t i = tid; i < A.items; i += step) gptr(A.itemC)[i] = 0;
  if (blockIdx.x) return;
  uint32_t* h[2] = {reinterpret_cast<uint32_t*>(A.inner), reinterpret_cast<uint32_t*>(A.whole)};
  for (uint32_t i = threadIdx.x; i < HEAD / 4; i += 256) gptr(h[0])[i] = gptr(h[1])[i] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    A.win[OUT] = A.W;
    A.inner->queue = reinterpret_cast<decltype(A.inner->queue)>(reinterpret_cast<char*>(A.inner) + HEAD - QUEUES);
    A.whole->queue = reinterpret_cast<decltype(A.whole->queue)>(reinterpret_cast<char*>(A.whole) + HEAD - QUEUES);
    nsgc_dev_plan* p = A.inner;
    p->gwin = A.win;
    p->gprefA = A.prefA;
    p->gitemB = A.itemB;
    p->goverB = A.goverB;
    p->goverW = A.goverW;
    p->num_grid = OUT;
    p->gitemsW = p->gitemsB = A.cells;
    p->gtile_log2 = TILE_LOG2;
    p->max_sweeps_log2 = 5;
    p->gmax_keys = 1u << 18;   // (sorting more takes one workgroup longer than all of them the window)
    p = A.whole;
    p->gwin = A.win + OUT;
    p->gitemC = A.itemC;
    p->goverC = A.goverC;
    p->num_grid = 1;
    p->gitemsC = A.items;
    p->gtile_log2 = TILE_LOG2;
    p->rc_slots_log2 = A.rc_slots_log2;
    p->max_sweeps_log2 = 5;
    p->out = A.out;
  }
}

// The outer cell of a packet, or OUT for one between two dominant addresses.
__device__ __forceinline__ uint32_t outer_cell(const nsgc_grid_desc& W, uint32_t r, uint32_t c, bool hs, bool hd) {
  if (hs && hd) return OUT;
  uint32_t i = r >> (32 - W.logA), j = c >> (32 - W.logBc);
  if (hs) i ^= strip_shift(c, W.logA);
  if (hd) j ^= strip_shift(r, W.logBc);
  return ((i >> W.subA) << OUT_LOG2) | (j >> W.subB);
}

// Packets of each outer cell in one range of the window, a workgroup each.
// Reads 8 bytes per packet; each wavefront counts in bins of its own.
constexpr uint32_t CNT_NT = 512;
__global__ __launch_bounds__(CNT_NT) void k_large_count(Args A) {
  constexpr uint32_t NW = CNT_NT / 64;
  __shared__ uint32_t idt[2 * HT];
  __shared__ uint32_t bins[NW][OUT];
  const uint32_t tid = threadIdx.x;
  const nsgc_grid_desc& W = A.W;
  const uint32_t sh = uniform(gptr(W.heavy)[2 * HV + HV * HV]), dh = uniform(gptr(W.heavy)[2 * HV + HV * HV + 1]);
  for (uint32_t i = tid; i < 2 * HT; i += CNT_NT) idt[i] = free_entry(i, i < HT ? sh : dh);
  for (uint32_t i = tid; i < NW * OUT; i += CNT_NT) (&bins[0][0])[i] = 0;
  __syncthreads();
  if (tid < 2 * HV) {
    const uint32_t id = gptr(W.heavy)[tid];
    if (id != EMPTY32) idt[(tid / HV) * HT + heavy_index(id, tid < HV ? sh : dh)] = id;
  }
  __syncthreads();
  uint32_t* const bin = bins[tid >> 6];
  const uint32_t beg = blockIdx.x * A.per * T, end = uint32_t(min(u64(W.n), u64(beg) + u64(A.per) * T));
  auto count = [&](uint32_t s, uint32_t d) {
    const uint32_t r = row_hash(s), c = col_hash(d);
    const uint32_t o = outer_cell(W, r, c, idt[heavy_index(r, sh)] == r, idt[HT + heavy_index(c, dh)] == c);
    if (o < OUT) lds_add(&bin[o], 1);
  };
  const NSGC_GLOBAL uint32_t* src = gptr(W.src);
  const NSGC_GLOBAL uint32_t* dst = gptr(W.dst);
  uint32_t at = beg;
  for (; end - at >= CNT_NT * 8; at += CNT_NT * 8) {   // (end >= at)
    v4u32 s4[2], d4[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      s4[k] = *(const NSGC_GLOBAL v4u32_any*)(src + at + (k * CNT_NT + tid) * 4);
      d4[k] = *(const NSGC_GLOBAL v4u32_any*)(dst + at + (k * CNT_NT + tid) * 4);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      count(s4[k].x, d4[k].x);
      count(s4[k].y, d4[k].y);
      count(s4[k].z, d4[k].z);
      count(s4[k].w, d4[k].w);
    }
  }
  for (at += tid; at < end; at += CNT_NT) count(src[at], dst[at]);
  __syncthreads();
  if (tid < OUT) {
    uint32_t x = 0;
#pragma unroll
    for (uint32_t k = 0; k < NW; ++k) x += bins[k][tid];
    gptr(A.cnt)[blockIdx.x * OUT + tid] = x;
  }
}

// Counts -> the position where each range's keys of each outer cell start, and
// the outer cells' windows.  One workgroup: four threads share an outer cell's
// column of counts.
__global__ __launch_bounds__(1024) void k_large_scan(Args A) {
  constexpr uint32_t PARTS = 1024 / OUT;
  __shared__ uint32_t part[PARTS][OUT];
  __shared__ uint32_t red[2][OUT / 64];
  const uint32_t cell = threadIdx.x & (OUT - 1), p = threadIdx.x / OUT;
  const uint32_t q = (A.ranges + PARTS - 1) / PARTS;
  const uint32_t beg = min(A.ranges, p * q), end = min(A.ranges, beg + q);
  NSGC_GLOBAL uint32_t* cnt = gptr(A.cnt) + cell;
  uint32_t x = 0;
#pragma unroll 16
  for (uint32_t i = beg; i < end; ++i) x += cnt[i * OUT];
  part[p][cell] = x;
  __syncthreads();
  uint32_t total = 0, before = 0;
  for (uint32_t k = 0; k < PARTS; ++k) {
    if (k < p) before += part[k][cell];
    total += part[k][cell];
  }
  // starts of the outer cells' regions and of their tiles
  const uint32_t tiles = (total + T - 1) / T;
  const uint32_t is = wave_inclusive_scan(total), it = wave_inclusive_scan(tiles);
  if (p == 0 && lane_id() == 63) {
    red[0][cell >> 6] = is;
    red[1][cell >> 6] = it;
  }
  __syncthreads();
  uint32_t base = is - total, first = it - tiles;
  for (uint32_t k = 0; k < (cell >> 6); ++k) {
    base += red[0][k];
    first += red[1][k];
  }
  uint32_t run = base + before;
  for (uint32_t i0 = beg; i0 < end; i0 += 16) {
    uint32_t y[16];
#pragma unroll
    for (uint32_t k = 0; k < 16; ++k) y[k] = i0 + k < end ? cnt[(i0 + k) * OUT] : 0u;
#pragma unroll
    for (uint32_t k = 0; k < 16; ++k) {
      if (i0 + k < end) cnt[(i0 + k) * OUT] = run;
      run += y[k];
    }
  }
  if (p) return;
  nsgc_grid_desc W = A.W;
  const uint32_t lg = W.subA + W.subB, sub = (1u << (W.logR - W.logA)) + (1u << (W.logC - W.logBc)) + 3;
  W.src = reinterpret_cast<const uint32_t*>(W.keys + base);
  W.dst = nullptr;
  W.keys = A.keys2 + base;
  W.tile = A.W.tile + (u64(first) << lg);
  W.rec = A.W.rec + (u64(cell) << lg) * sub;
  W.acc = A.acc + (u64(cell) << lg) * (2 * HV);
  W.partB = A.partB + (u64(cell) << lg) * 4;
  W.partC = nullptr;
  W.n = total;
  W.ntiles = tiles;
  W.itemB = cell << lg;
  W.itemC = 0;
  W.base = base;
  W.strip_i = uint16_t((cell >> OUT_LOG2) << W.subA);
  W.strip_j = uint16_t((cell & ((1u << OUT_LOG2) - 1u)) << W.subB);
  A.win[cell] = W;
  gptr(A.prefA)[cell] = first;
  if (cell == OUT - 1) {
    gptr(A.prefA)[OUT] = first + tiles;
    A.inner->gitemsA = first + tiles;
  }
}

// Keys into their outer cells' regions, tile by tile: a tile's keys are placed
// in LDS by outer cell and leave in runs, a wavefront per run.  One workgroup
// takes a contiguous part of the ranges, so that its positions carry on from
// tile to tile and its share of the matrix is added to memory once.
constexpr uint32_t SP_NT = 1024;
constexpr uint32_t SP_PER = T / SP_NT;
constexpr size_t split_lds() { return size_t(T) * 8 + (2 * OUT + 4 + HV * HV + 2 * HT) * 4 + 2 * HT + 64; }
__global__ __launch_bounds__(SP_NT) void k_large_split(Args A) {
  extern __shared__ __align__(16) unsigned char smem[];
  u64* stage = reinterpret_cast<u64*>(smem);                   // [T]
  uint32_t* hist = reinterpret_cast<uint32_t*>(stage + T);     // [OUT + 1] counts, then starts
  uint32_t* cursor = hist + OUT + 4;                           // [OUT] next position of each outer cell
  uint32_t* mat = cursor + OUT;                                // [HV][HV]
  uint32_t* idt = mat + HV * HV;                               // [2][HT]
  uint8_t* ids = reinterpret_cast<uint8_t*>(idt + 2 * HT);     // [2][HT]
  uint32_t* red = reinterpret_cast<uint32_t*>(ids + 2 * HT);   // [OUT / 64]
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = lane_id();
  const nsgc_grid_desc& W = A.W;
  const uint32_t q = (A.ranges + gridDim.x - 1) / gridDim.x;
  const uint32_t r0 = min(A.ranges, blockIdx.x * q), r1 = min(A.ranges, r0 + q);
  if (r0 >= r1) return;
  const uint32_t tiles = (W.n + T - 1) / T;
  const uint32_t t0 = r0 * A.per, t1 = min(tiles, r1 * A.per);
  uint32_t r[SP_PER], c[SP_PER];
  auto load = [&](uint32_t t) {
    const NSGC_GLOBAL uint32_t* src = gptr(W.src) + t * T;
    const NSGC_GLOBAL uint32_t* dst = gptr(W.dst) + t * T;
    const uint32_t len = min(T, W.n - t * T);
    if (len == T) {
#pragma unroll
      for (uint32_t k = 0; k < SP_PER / 4; ++k) {
        const uint32_t at = (k * SP_NT + tid) * 4;
        const v4u32 s4 = *(const NSGC_GLOBAL v4u32_any*)(src + at);
        const v4u32 d4 = *(const NSGC_GLOBAL v4u32_any*)(dst + at);
        r[4 * k + 0] = s4.x; r[4 * k + 1] = s4.y; r[4 * k + 2] = s4.z; r[4 * k + 3] = s4.w;
        c[4 * k + 0] = d4.x; c[4 * k + 1] = d4.y; c[4 * k + 2] = d4.z; c[4 * k + 3] = d4.w;
      }
    } else {
#pragma unroll
      for (uint32_t k = 0; k < SP_PER; ++k) {
        const uint32_t at = min(((k >> 2) * SP_NT + tid) * 4 + (k & 3), len - 1);
        r[k] = src[at];
        c[k] = dst[at];
      }
    }
  };
  load(t0);
  const uint32_t sh = uniform(gptr(W.heavy)[2 * HV + HV * HV]), dh = uniform(gptr(W.heavy)[2 * HV + HV * HV + 1]);
  for (uint32_t i = tid; i < 2 * HT; i += SP_NT) idt[i] = free_entry(i, i < HT ? sh : dh);
  for (uint32_t i = tid; i < HV * HV; i += SP_NT) mat[i] = 0;
  if (tid < OUT) {
    hist[tid] = 0;
    cursor[tid] = gptr(A.cnt)[r0 * OUT + tid];
  }
  lds_barrier();
  if (tid < 2 * HV) {
    const uint32_t id = gptr(W.heavy)[tid];
    if (id != EMPTY32) {
      const uint32_t at = (tid / HV) * HT + heavy_index(id, tid < HV ? sh : dh);
      idt[at] = id;
      ids[at] = uint8_t(tid & (HV - 1));
    }
  }
  lds_barrier();
  for (uint32_t t = t0; t < t1; ++t) {
    const uint32_t len = min(T, W.n - t * T);
    uint32_t br[SP_PER];   // rank in its outer cell << 8 | outer cell; all ones: no key
#pragma unroll
    for (uint32_t k = 0; k < SP_PER; ++k) {
      r[k] = row_hash(r[k]);
      c[k] = col_hash(c[k]);
      const bool hs = idt[heavy_index(r[k], sh)] == r[k], hd = idt[HT + heavy_index(c[k], dh)] == c[k];
      const bool ok = len == T || ((k >> 2) * SP_NT + tid) * 4 + (k & 3) < len;
      const uint32_t o = outer_cell(W, r[k], c[k], hs, hd);
      br[k] = ~0u;
      if (ok) {
        if (o == OUT) lds_add(&mat[uint32_t(ids[heavy_index(r[k], sh)]) * HV + ids[HT + heavy_index(c[k], dh)]], 1);
        else br[k] = (lds_add(&hist[o], 1) << 8) | o;
      }
    }
    lds_barrier();
    uint32_t mine = 0, incl = 0;
    if (tid < OUT) {   // counts -> starts
      mine = hist[tid];
      incl = wave_inclusive_scan(mine);
      if (lane == 63) red[w] = incl;
    }
    lds_barrier();
    if (tid < OUT) {
      uint32_t s = incl - mine;
      for (uint32_t k = 0; k < w; ++k) s += red[k];
      hist[tid] = s;
      if (tid == OUT - 1) hist[OUT] = s + mine;
    }
    lds_barrier();
#pragma unroll
    for (uint32_t k = 0; k < SP_PER; ++k)
      if (br[k] != ~0u) stage[hist[br[k] & (OUT - 1)] + (br[k] >> 8)] = (u64(r[k]) << 32) | c[k];
    lds_barrier();
    if (t + 1 < t1) load(t + 1);
    NSGC_GLOBAL u64* keys = gptr(W.keys);
    for (uint32_t o = w; o < OUT; o += SP_NT / 64) {
      const uint32_t s = uniform(hist[o]), e = uniform(hist[o + 1]), to = uniform(cursor[o]);
      for (uint32_t k = lane; k < e - s; k += 64) keys[u64(to) + k] = stage[s + k];
      if (lane == 0) cursor[o] = to + (e - s);
    }
    lds_barrier();
    if (tid < OUT) hist[tid] = 0;
    lds_barrier();
  }
  NSGC_GLOBAL uint32_t* m = gptr(W.heavy) + 2 * HV;
  for (uint32_t i = tid; i < HV * HV; i += SP_NT)
    if (mat[i]) __hip_atomic_fetch_add(m + i, mat[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Totals and dominant counters of an outer cell's cells, a workgroup each.
__global__ __launch_bounds__(512) void k_large_reduce(Args A) {
  __shared__ u64 sum[512];
  __shared__ uint32_t red[8][4];
  const uint32_t tid = threadIdx.x, o = blockIdx.x, cells = 1u << (A.W.subA + A.W.subB);
  const NSGC_GLOBAL u64* acc = gptr(A.acc) + u64(o) * cells * (2 * HV);
  u64 x = 0;
#pragma unroll 8
  for (uint32_t i = tid; i < cells * 2 * HV; i += 512) x += acc[i];
  sum[tid] = x;
  const NSGC_GLOBAL v4u32* pb = gptr(reinterpret_cast<const v4u32*>(A.partB)) + u64(o) * cells;
  uint32_t packets = 0, links = 0, mx = 0, bad = 0;
  for (uint32_t i = tid; i < cells; i += 512) {
    const v4u32 y = pb[i];
    packets += y.x;
    links += y.y;
    mx = max(mx, y.z);
    bad |= y.w;
  }
  packets = wave_sum(packets);
  links = wave_sum(links);
  mx = wave_max(mx);
  bad = wave_max(bad);
  if (lane_id() == 0) {
    red[tid >> 6][0] = packets;
    red[tid >> 6][1] = links;
    red[tid >> 6][2] = mx;
    red[tid >> 6][3] = bad;
  }
  __syncthreads();
  if (tid < 2 * HV) {
    for (uint32_t k = 2 * HV; k < 512; k += 2 * HV) x += sum[k + tid];
    gptr(A.W.acc)[o * (2 * HV) + tid] = x;
  }
  if (tid == 0) {
    for (uint32_t k = 1; k < 8; ++k) {
      packets += red[k][0];
      links += red[k][1];
      mx = max(mx, red[k][2]);
      bad |= red[k][3];
    }
    const v4u32 part = {packets, links, mx, bad};
    gptr(reinterpret_cast<v4u32*>(A.W.partB))[o] = part;
  }
}

}  // namespace

size_t large_grid_bytes(unsigned long long n) {
  Shape g;
  return shape(n, &g) ? g.total : 0;
}

hipError_t large_grid_allow_lds(size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_large_split),
                             hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
}

hipError_t large_grid_stats(const uint32_t* src, const uint32_t* dst, unsigned long long n, void* ws,
                            unsigned long long* out, const LargeGridLaunch& L, hipStream_t s) {
  Shape g;
  if (!shape(n, &g)) return hipErrorInvalidValue;
  char* const base = static_cast<char*>(ws);
  auto words = [&](size_t at) { return reinterpret_cast<uint32_t*>(base + at); };
  auto longs = [&](size_t at) { return reinterpret_cast<unsigned long long*>(base + at); };
  Args A = {};
  A.W.src = src;
  A.W.dst = dst;
  A.W.keys = longs(0);
  A.W.emit_row = longs(0);   // (the outer cells' keys have been partitioned when entries are emitted)
  A.W.emit_col = longs(g.emit_col);
  A.W.tile = words(g.tile);
  A.W.rec = words(g.rec);
  A.W.heavy = words(g.heavy);
  A.W.acc = longs(g.acc2);
  A.W.partB = words(g.partB2);
  A.W.partC = words(g.partC);
  A.W.n = uint32_t(n);
  A.W.logA = uint8_t(g.a);
  A.W.logBc = uint8_t(g.b);
  A.W.logR = uint8_t(g.logR);
  A.W.logC = uint8_t(g.logC);
  A.W.subA = uint8_t(g.a - OUT_LOG2);
  A.W.subB = uint8_t(g.b - OUT_LOG2);
  A.W.logRi = uint8_t(g.logRi);
  A.W.logCi = uint8_t(g.logCi);
  A.W.logP = 2 * OUT_LOG2;
  A.win = reinterpret_cast<nsgc_grid_desc*>(base + g.win);
  A.inner = reinterpret_cast<nsgc_dev_plan*>(base + g.head);
  A.whole = reinterpret_cast<nsgc_dev_plan*>(base + g.head + HEAD);
  A.cnt = words(g.cnt);
  A.prefA = words(g.prefA);
  A.itemB = words(g.itemB);
  A.itemC = words(g.itemC);
  A.goverB = words(g.goverB);
  A.goverW = words(g.goverW);
  A.goverC = words(g.goverC);
  A.keys2 = longs(g.keys2);
  A.acc = longs(g.acc);
  A.partB = words(g.partB);
  A.out = out;
  A.cells = g.cells;
  A.items = g.items;
  A.per = g.per;
  A.ranges = g.ranges;
  A.rc_slots_log2 = L.rc_slots_log2;
  hipError_t e;
  hipLaunchKernelGGL(k_large_init, dim3(64), dim3(256), 0, s, A);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_grid_heavy(A.whole, TILE_LOG2, 1, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_large_count, dim3(g.ranges), dim3(CNT_NT), 0, s, A);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_large_scan, dim3(1), dim3(1024), 0, s, A);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_large_split, dim3(std::min(g.ranges, L.cus)), dim3(SP_NT), split_lds(), s, A);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_grid_partition(A.inner, TILE_LOG2, 1u << NSGC_GRID_MAX_CELLS_LOG2, L.cus, s, true)) !=
      hipSuccess)
    return e;
  if ((e = launch_grid_links(A.inner, 1, L.links, s)) != hipSuccess) return e;
  if ((e = launch_grid_links(A.inner, 2, L.wide, s)) != hipSuccess) return e;
  if ((e = launch_grid_rounds(A.inner, true, L.rounds, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_large_reduce, dim3(OUT), dim3(512), 0, s, A);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_grid_rowcol(A.whole, L.rowcol, L.lds_rowcol, s)) != hipSuccess) return e;
  if ((e = launch_grid_sweeps(A.whole, L.sweeps, L.lds_sweeps, s)) != hipSuccess) return e;
  return launch_grid_finish(A.whole, s);
}

}  // namespace nsgc
