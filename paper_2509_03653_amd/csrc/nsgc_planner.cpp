// Host planner (see nsgc_plan.h for the tiers and phases it lays out).
#include "nsgc_planner.hpp"

#include "nsgc_large.hpp"

#include <algorithm>
#include <cstring>

namespace nsgc {

namespace {

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// A pointer field of a device descriptor.
template <class T>
T* at(uint64_t address) {
  return reinterpret_cast<T*>(address);
}
template <class T>
void rebase(T*& field, uint64_t base) {
  field = reinterpret_cast<T*>(reinterpret_cast<uint64_t>(field) + base);
}

// Whether a window of n packets above small_max is still taken whole by one
// workgroup: up to eight times small_max, as far as its tables go, unless the
// tuning asks for a form that only the partitioned kernels have.  (At 8192
// packets one workgroup takes 33 us and the partitioned kernels 47; above, the
// grid's tables spread over the chip.)
bool whole_window(uint64_t n, bool entity, const nsgc_tune& tune, const nsgc_tune_class& tc) {
  return !entity && n <= std::min<uint64_t>(8 * uint64_t(tune.small_max), NSGC_WHOLE_D) && tc.wave_target > 0 &&
         tune.combine_probes == 0 && !tune.row_complete;
}

// The size of the kernel it takes (n <= NSGC_WHOLE_D; small_max is at most 2048).
int whole_size(uint64_t n) {
  return n <= NSGC_WHOLE_A ? 0 : n <= NSGC_WHOLE_B ? 1 : n <= NSGC_WHOLE_C ? 2 : 3;
}

// Packets of a row or column bucket of the entity lists, at most.
constexpr uint64_t kListBucket = 1740;

// Workgroups of each size that 256 compute units hold at once.
constexpr size_t kWholeRound[NSGC_WHOLE] = {6144, 1536, 768, 256};

// Whether a window of n packets can be a grid window, and its grid (from
// NSGC_GRID_MIN packets on by right; shorter ones may ride along).  Cells hold four wavefront
// targets of packets, up to the cap on link buckets; the grid has four or more
// strips each way (with fewer, a dominant address cannot be spread) and as
// many row strips as row buckets if it can, since a strip of one bucket needs
// no counting.
bool grid_window(uint64_t n, bool entity, int finer, const nsgc_tune& tune, const nsgc_tune_class& tc,
                 nsgc_grid_desc* g) {
  if (tc.wave_target <= 0 || tune.combine_probes > 0 || n < (entity ? NSGC_GRID_ENTITY : NSGC_GRID_RIDE)) return false;
  const bool ride = n < NSGC_GRID_MIN;
  const uint64_t target = 4 * uint64_t(tc.wave_target);
  const int lc = std::min(std::min(ride ? 4 : ceil_log2((n + target - 1) / target) + finer,
                                   int(tune.max_link_buckets_log2)), NSGC_GRID_MAX_CELLS_LOG2);
  // Row and column buckets of at most NSGC_GRID_BUCKET packets: phase C takes
  // one and a half times as many entries in a single pass, and a bucket has at
  // most as many entries as packets.
  const auto buckets = [&](int32_t tuned) {
    const uint64_t t = std::min<uint64_t>(uint64_t(tuned), NSGC_GRID_BUCKET);
    return ceil_log2((n + t - 1) / t);
  };
  int logR = ride ? 2 : buckets(tc.row_target), logC = ride ? 2 : buckets(tc.col_target);
  const int a = std::min(std::min(logR, NSGC_GRID_MAX_A), lc - 2);
  const int b = std::min(std::min(lc - a, logC), NSGC_GRID_MAX_B);
  if (a < 2 || b < 2 || (entity && std::max(a, b) > std::min(a, b) + NSGC_GRID_MAX_SUB_LOG2)) return false;
  logR = std::min(logR, a + NSGC_GRID_MAX_SUB_LOG2);
  logC = std::min(logC, b + NSGC_GRID_MAX_SUB_LOG2);
  if (entity) logR = logC = std::max(std::min(logR, logC), std::max(a, b));   // merged phase-C items
  std::memset(g, 0, sizeof *g);
  g->n = uint32_t(n);
  g->logA = uint8_t(a);
  g->logBc = uint8_t(b);
  g->subA = g->logA;
  g->subB = g->logBc;
  g->logP = uint8_t(a + b);
  g->logR = uint8_t(logR);
  g->logC = uint8_t(logC);
  // A phase-C item takes one bucket in windows below 2^19 packets, two below 2^20
  // and four in larger ones, which have fewer links per packet; it splits them
  // again where they do not fit one pass.  (Eight windows of 2^19 packets among
  // 4096 addresses, nearly all distinct links: 168 us with four buckets per item,
  // 157 with two; 16 heavy-tailed ones 220 and 198; 16 of 2^21 with a dominant
  // address 444 with four and 458 with two.)
  const int gi = entity || n < (uint64_t(1) << 19) ? 0 : n < (uint64_t(1) << 20) ? 1 : 2;
  g->logRi = uint8_t(std::max(logR - gi, a));
  g->logCi = uint8_t(std::max(logC - gi, b));
  return true;
}

// A batch of fewer packets leaves compute units idle with full cells, and each
// cell is a serial chain: it takes up to four times as many.  (One window of
// 2^17 packets: 45 us with 128 cells, 38 with 512, 48 with 1024; of 2^18 49, 43
// with 512 and 51 with 1024; eight windows of 2^17 do not care.)
constexpr uint64_t kFinerPackets = uint64_t(512) << 10;
constexpr int kFinerMost = 2;

// The kernel of a grid window's phase B (0 SMALL, 1 BIG, 2 WIDE): a 2048-slot
// table would be more than half full above 1280 packets per cell, and above 4096
// BIG would leave most cells to WIDE after a reading of its own (one window of
// 1.2 * 10^7 packets among 4096 addresses 0.74 -> 0.69 ms without it).
int grid_kind(const nsgc_grid_desc& g) {
  const uint32_t cells = g.logA + g.logBc;
  return g.n > uint64_t(NSGC_GRID_BIG_KEYS) << cells ? 2 : g.n >> cells > NSGC_GRID_SMALL_CELLS ? 1 : 0;
}

// Partition tile (log2).  Tiles of 2^14 packets where a window has more than
// 1024 cells (their runs of keys per cell are longer); else 2^13, of which two
// fit a compute unit and overlap; smaller ones, down to 2^11, as long as the
// batch has fewer than two tiles per compute unit and its longest window few;
// and larger ones than the tuning's if SMALL's or BIG's longest window would
// have more tiles than their threads take.
constexpr uint64_t kGridTiles = 512;
uint32_t grid_tile_log2(uint64_t packets, uint32_t cells, const uint32_t (&longest)[3], const nsgc_tune& tune) {
  uint32_t k = uint32_t(tune.tile_log2);
  if (cells > NSGC_GRID_TILE13_CELLS) return 14;
  k = std::min(k, 13u);
  const uint32_t most = std::max(std::max(longest[0], longest[1]), longest[2]);
  while (k > 11 && (packets >> k) < kGridTiles && (most >> k) < NSGC_GRID_SMALL_TILES / 2) --k;
  const auto tiles = [&](int kind) { return (uint64_t(longest[kind]) + (uint64_t(1) << k) - 1) >> k; };
  while (tiles(0) > NSGC_GRID_SMALL_TILES || tiles(1) > NSGC_GRID_BIG_TILES) ++k;
  return k;
}
// (up to 1280 and 4096 packets in each of 1024 cells: 2^13-packet tiles do)
static_assert(NSGC_GRID_TILE13_CELLS * (NSGC_GRID_SMALL_CELLS + 1) <= NSGC_GRID_SMALL_TILES << 13, "SMALL");
static_assert(NSGC_GRID_TILE13_CELLS * NSGC_GRID_BIG_KEYS <= NSGC_GRID_BIG_TILES << 13, "BIG");
static_assert((NSGC_GRID_BIG_KEYS << NSGC_GRID_MAX_CELLS_LOG2) <= NSGC_GRID_BIG_TILES << 14, "BIG, large tiles");

}  // namespace

uint32_t grid_max_cells(uint32_t tile_log2) {
  return tile_log2 >= 14 ? 1u << NSGC_GRID_MAX_CELLS_LOG2 : NSGC_GRID_TILE13_CELLS;
}

int ceil_log2(uint64_t x) {
  int k = 0;
  while ((uint64_t(1) << k) < x) ++k;
  return k;
}

void default_tune(nsgc_tune* t) {
  std::memset(t, 0, sizeof(*t));
  t->small_max = 1024;
  t->tile_log2 = 14;
  t->link_slots_log2 = 12;
  t->rc_slots_log2 = 12;
  t->blocks_per_cu = 3;
  t->max_link_buckets_log2 = 11;
  t->max_rc_buckets_log2 = 10;
  t->max_sweeps_log2 = 24;
  t->combine_probes = 0;
  t->large_min_log2 = 24;
  t->row_complete = 0;
  // Per size class (windows of [2^k, 2^(k+1)) packets): below 2^23 packets a
  // link bucket holds at most as many packets as its LDS table has slots (at
  // 2^23, twice as many), so it sweeps only when nearly all its packets are
  // distinct links.  A row or column bucket of a window of 2^19 packets or
  // more holds up to four times as many packets as its table has slots: its
  // ids are distinct sources (destinations), of which large windows of
  // heavy-tailed traffic have far fewer than packets (2^23-packet windows
  // measured 0.03-0.1 distinct ids per packet), and the larger phase-C items
  // and longer phase-B segments measured 11% faster per batch than twice as
  // many buckets.  Windows below 2^19 packets keep the smaller buckets, which
  // measured faster there.  (That is for one link bucket per hash range; grid
  // windows take buckets of up to 4096 packets and cells of four wavefront
  // targets.)
  for (int k = 0; k <= 32; ++k) {
    nsgc_tune_class& c = t->cls[k];
    c.link_target = k < 19 ? 2048 : k < 23 ? 4096 : 8192;
    c.row_target = c.col_target = k < 19 ? 4096 : 16384;
    c.wave_target = 256;
  }
}

int check_tune(const nsgc_tune& t) {
  if (t.small_max < 0 || t.small_max > 2048) return NSGC_ERR_INVALID_ARG;
  if (t.tile_log2 < 11 || t.tile_log2 > 14) return NSGC_ERR_INVALID_ARG;
  if (t.link_slots_log2 < 10 || t.link_slots_log2 > 12) return NSGC_ERR_INVALID_ARG;
  if (t.rc_slots_log2 < 10 || t.rc_slots_log2 > 13) return NSGC_ERR_INVALID_ARG;
  if (t.blocks_per_cu < 1 || t.blocks_per_cu > 16) return NSGC_ERR_INVALID_ARG;
  if (t.max_link_buckets_log2 < 0 || t.max_link_buckets_log2 > 12) return NSGC_ERR_INVALID_ARG;
  if (t.max_rc_buckets_log2 < 0 || t.max_rc_buckets_log2 > 12) return NSGC_ERR_INVALID_ARG;
  if (t.max_sweeps_log2 < 0 || t.max_sweeps_log2 > 24) return NSGC_ERR_INVALID_ARG;
  if (t.combine_probes < 0 || t.combine_probes > 64) return NSGC_ERR_INVALID_ARG;
  if (t.large_min_log2 < 20 || t.large_min_log2 > 33) return NSGC_ERR_INVALID_ARG;
  if (t.row_complete < 0 || t.row_complete > 1) return NSGC_ERR_INVALID_ARG;
  for (int k = 0; k <= 32; ++k) {
    const nsgc_tune_class& c = t.cls[k];
    if (c.link_target < 64 || c.row_target < 64 || c.col_target < 64) return NSGC_ERR_INVALID_ARG;
    if (c.wave_target != 0 && (c.wave_target < 64 || c.wave_target > 2048)) return NSGC_ERR_INVALID_ARG;
  }
  return NSGC_OK;
}

int validate_offsets(const int64_t* offsets, int64_t num_windows) {
  if (offsets[0] < 0) return NSGC_ERR_BAD_OFFSETS;
  for (int64_t w = 0; w < num_windows; ++w) {
    const int64_t n = offsets[w + 1] - offsets[w];
    if (offsets[w + 1] < offsets[w]) return NSGC_ERR_BAD_OFFSETS;
    if (n > int64_t(0xFFFFFFFFll)) return NSGC_ERR_BAD_OFFSETS;
  }
  return NSGC_OK;
}

int make_plan(const int64_t* offsets, int64_t num_windows, const nsgc_tune& tune,
              HostPlan* p, bool entity, bool allow_large, bool allow_grid) {
  p->large.clear();
  p->large_max = 0;
  p->entity = entity;
  p->ent_cur.clear();
  p->ent_end.clear();
  p->small.clear();
  p->win.clear();
  p->prefA.clear();
  p->prefB.clear();
  p->prefC.clear();
  p->itemwinB.clear();
  p->itemwinC.clear();
  p->mapBb.clear();
  p->mapBw.clear();
  p->shape.clear();
  p->gwin.clear();
  p->gprefA.clear();
  p->gitemB.clear();
  p->gitemC.clear();
  std::vector<nsgc_small_desc> whole[NSGC_WHOLE];   // windows taken whole, by size
  std::vector<nsgc_grid_desc> grid[3];      // grid windows by the kernel of their phase B
  uint64_t gpackets = 0;
  uint32_t glongest[3] = {0, 0, 0};
  uint32_t gcells = 0;   // most cells of a grid window
  p->itemsBb = p->itemsBw = 0;
  p->wave_rc_max = 0;
  p->num_rows = 0;
  p->tier.assign(size_t(num_windows), 0);
  p->ws_elems = p->tilemeta_words = p->lbmeta_words = 0;
  p->tile_log2 = uint32_t(tune.tile_log2);
  p->link_slots_log2 = uint32_t(tune.link_slots_log2);
  p->rc_slots_log2 = uint32_t(tune.rc_slots_log2);
  p->max_sweeps_log2 = uint32_t(tune.max_sweeps_log2);
  p->combine_probes = uint32_t(tune.combine_probes);
  p->small_slots_log2 = uint32_t(std::max(ceil_log2(uint64_t(std::max(tune.small_max, 1)) * 2), 6));

  const uint64_t tile = uint64_t(1) << tune.tile_log2;
  uint64_t a = 0, b = 0, c = 0;
  const uint64_t packets = num_windows > 0 ? uint64_t(offsets[num_windows] - offsets[0]) : 0;
  int finer = 0;
  while (finer < kFinerMost && (packets << finer) < kFinerPackets) ++finer;
  for (int64_t w = 0; w < num_windows; ++w) {
    const uint64_t n = uint64_t(offsets[w + 1] - offsets[w]);
    if (n <= uint64_t(tune.small_max)) {
      nsgc_small_desc s;
      s.in_begin = offsets[w];
      s.n = uint32_t(n);
      s.out_index = uint32_t(w);
      (entity ? p->small : whole[whole_size(n)]).push_back(s);
      p->tier[size_t(w)] = n == 0 ? 0 : 1;
      continue;
    }
    if (allow_large && !entity && tune.large_min_log2 < 33 &&
        n >= (uint64_t(1) << tune.large_min_log2)) {
      p->large.push_back({offsets[w], n, uint32_t(w)});
      p->large_max = std::max(p->large_max, n);
      p->tier[size_t(w)] = 3;
      continue;
    }
    p->tier[size_t(w)] = 2;
    int cls = 0;
    while (cls < 32 && (uint64_t(1) << (cls + 1)) <= n) ++cls;
    const nsgc_tune_class& tc = tune.cls[cls];
    const int capB = tune.max_link_buckets_log2, capRC = tune.max_rc_buckets_log2;
    nsgc_win_desc d;
    std::memset(&d, 0, sizeof d);
    d.in_begin = offsets[w];
    d.n = uint32_t(n);
    d.out_index = uint32_t(w);
    d.logB = uint8_t(std::min(ceil_log2((n + uint64_t(tc.link_target) - 1) / uint64_t(tc.link_target)), capB));
    d.logR = uint8_t(std::min(ceil_log2((n + uint64_t(tc.row_target) - 1) / uint64_t(tc.row_target)), capRC));
    d.logC = uint8_t(std::min(ceil_log2((n + uint64_t(tc.col_target) - 1) / uint64_t(tc.col_target)), capRC));
    if (entity) d.logR = d.logC = std::max(d.logR, d.logC);   // merged phase-C items
    if (entity && !allow_grid) {
      // The lists' table of 4096 slots holds the addresses of both views, as many
      // as packets and more where all are distinct: buckets of up to 1740 packets
      // (of 4096 it takes several sweeps, twice; see k_rowcol_ent), as far as a
      // wavefront's counters go.
      const int fine = ceil_log2((n + kListBucket - 1) / kListBucket);
      d.logR = d.logC = uint8_t(std::max<int>(d.logR, std::min({fine, capRC, ceil_log2(NSGC_WAVE_MAX_RC)})));
    }
    // one wavefront per link bucket when the window's buckets fit its tables
    if (tc.wave_target > 0 && (1u << d.logR) <= NSGC_WAVE_MAX_RC && (1u << d.logC) <= NSGC_WAVE_MAX_RC) {
      const int lw = ceil_log2((n + uint64_t(tc.wave_target) - 1) / uint64_t(tc.wave_target));
      if (lw <= capB) {
        d.logB = uint8_t(lw);
        d.wave = 1;
      }
    }
    p->shape.push_back({d.logB, d.logR, d.logC, int64_t((n + tile - 1) / tile)});
    if (whole_window(n, entity, tune, tc)) {
      whole[whole_size(n)].push_back({offsets[w], uint32_t(n), uint32_t(w)});
      continue;
    }
    nsgc_grid_desc g;
    if (allow_grid && !(tune.row_complete && d.wave) &&
        (entity ? capB >= 4 && capRC >= 2 : n >= NSGC_GRID_MIN && d.logR >= 2 && d.logC >= 2) &&
        grid_window(n, entity, finer, tune, tc, &g)) {
      g.src = at<uint32_t>(uint64_t(offsets[w]) * 4);   // byte offsets until serialize()
      g.out_index = uint32_t(w);
      const int kind = grid_kind(g);
      grid[kind].push_back(g);
      gpackets += n;
      glongest[kind] = std::max(glongest[kind], uint32_t(n));
      gcells = std::max(gcells, 1u << (g.logA + g.logBc));
      continue;
    }
    if (d.wave) p->wave_rc_max = std::max(p->wave_rc_max, 1u << std::max(d.logR, d.logC));
    // row-complete: wavefront windows of two or more link buckets
    if (tune.row_complete && d.wave && !entity && d.logB >= 1) {
      d.rows = 1;
      ++p->num_rows;
    }
    d.ntiles = uint32_t((n + tile - 1) / tile);
    d.counter = uint32_t(p->win.size());
    d.ws = p->ws_elems;
    d.tilemeta = p->tilemeta_words;
    d.lbmeta = p->lbmeta_words;
    const uint64_t B = uint64_t(1) << d.logB, R = uint64_t(1) << d.logR, C = uint64_t(1) << d.logC;
    p->ws_elems += int64_t(n);
    p->tilemeta_words += int64_t(uint64_t(d.ntiles) * (B + 1));
    p->lbmeta_words += int64_t(B * (R + C + 3));
    p->prefA.push_back(uint32_t(a));
    p->prefB.push_back(uint32_t(b));
    p->prefC.push_back(uint32_t(c));
    const uint32_t wi = uint32_t(p->win.size());
    p->itemwinB.insert(p->itemwinB.end(), size_t(B), wi);
    std::vector<uint32_t>& m = d.wave ? p->mapBw : p->mapBb;
    for (uint64_t i = 0; i < B; ++i) m.push_back(uint32_t(b + i));
    p->itemwinC.insert(p->itemwinC.end(), size_t(R + C), wi);
    a += d.ntiles;
    b += B;
    c += R + C;
    if (a > 0xFFFFFFFFull || b > 0xFFFFFFFFull || c > 0xFFFFFFFFull) return NSGC_ERR_INVALID_ARG;
    p->win.push_back(d);
  }
  // Beside grid windows up to NSGC_GRID_RIDERS of the longer ones join them, and
  // all of them if that spares their launch, which stands in front of a small
  // batch's chain of kernels (windows of 20698 and 7074 packets: 67 us apart, 48
  // on the grid; 7 of 1947 .. 22721: 60 and 42; 45 of 1143 .. 16547: 69 and 51;
  // but 1500 of 2700 .. 13858: 322 and 376).
  if (gpackets) {
    const bool all = whole[0].empty() && whole[1].empty() && whole[2].size() + whole[3].size() <= NSGC_GRID_RIDERS;
    size_t riders = 0;
    for (int k = 2; k < NSGC_WHOLE; ++k) {
      std::vector<nsgc_small_desc> stay;
      for (const nsgc_small_desc& s : whole[k]) {
        nsgc_grid_desc g;
        if (riders == NSGC_GRID_RIDERS || (!all && s.n < NSGC_GRID_RIDE_APART) ||
            !grid_window(s.n, false, 0, tune, tune.cls[ceil_log2(s.n + 1) - 1], &g)) {
          stay.push_back(s);
          continue;
        }
        ++riders;
        g.src = at<uint32_t>(uint64_t(s.in_begin) * 4);
        g.out_index = s.out_index;
        gpackets += g.n;
        grid[0].push_back(g);
      }
      whole[k].swap(stay);
    }
  }
  // A launch more costs 6 to 10 us: sizes that fit the chip at once in a larger
  // size's kernel go there (180 windows of 6 .. 524 packets: 25 us in two
  // launches, 15 in one).
  for (int k = 0; k < NSGC_WHOLE; ++k) {
    int next = k + 1;
    while (next < NSGC_WHOLE && whole[next].empty()) ++next;
    if (next < NSGC_WHOLE && whole[k].size() + whole[next].size() <= kWholeRound[next]) {
      whole[next].insert(whole[next].end(), whole[k].begin(), whole[k].end());
      whole[k].clear();
    }
    p->num_whole[k] = uint32_t(whole[k].size());
    p->small.insert(p->small.end(), whole[k].begin(), whole[k].end());
  }
  // grid windows: tile size, then tiles, cells and phase-C items in order
  p->gtile_log2 = grid_tile_log2(gpackets, gcells, glongest, tune);
  for (const std::vector<nsgc_grid_desc>& g : grid) p->gwin.insert(p->gwin.end(), g.begin(), g.end());
  const size_t nsmall = grid[0].size(), nbig = nsmall + grid[1].size();
  uint64_t ga = 0, gb = 0, gc = 0;
  p->gtile_words = p->grec_words = 0;
  p->gitemsS = p->gitemsW = 0;
  p->gbuckets = 0;
  for (size_t i = 0; i < p->gwin.size(); ++i) {
    nsgc_grid_desc& g = p->gwin[i];
    g.ntiles = uint32_t((uint64_t(g.n) + (uint64_t(1) << p->gtile_log2) - 1) >> p->gtile_log2);
    const uint64_t cells = uint64_t(1) << (g.logA + g.logBc);
    const uint64_t R = uint64_t(1) << g.logR, C = uint64_t(1) << g.logC;
    const uint64_t hv = NSGC_GRID_HV(p->gtile_log2);
    const uint64_t items = (uint64_t(1) << g.logRi) + (entity ? 0 : uint64_t(1) << g.logCi) + NSGC_GRID_CITEMS(hv);
    g.keys = at<unsigned long long>(uint64_t(p->ws_elems) * 8);
    g.tile = at<uint32_t>(uint64_t(p->gtile_words) * 4);
    g.rec = at<uint32_t>(uint64_t(p->grec_words) * 4);
    g.heavy = at<uint32_t>(i * NSGC_GRID_HV_WORDS(hv) * 4);
    g.acc = at<unsigned long long>(gb * 2 * hv * 8);
    g.partB = at<uint32_t>(gb * 16);
    g.partC = at<uint32_t>(gc * 16);
    g.itemB = uint32_t(gb);
    g.itemC = uint32_t(gc);
    p->ws_elems += int64_t(g.n);
    p->gtile_words += int64_t(uint64_t(g.ntiles) * cells);
    p->grec_words += int64_t(cells * ((R >> g.logA) + (C >> g.logBc) + 3));
    p->gprefA.push_back(uint32_t(ga));
    p->gitemB.insert(p->gitemB.end(), size_t(cells), uint32_t(i));
    p->gitemC.insert(p->gitemC.end(), size_t(items), uint32_t(i));
    p->gbuckets += uint32_t(R + C);
    ga += g.ntiles;
    gb += cells;
    gc += items;
    if (ga > 0xFFFFFFFFull || gb > 0xFFFFFFFFull || gc > 0xFFFFFFFFull) return NSGC_ERR_INVALID_ARG;
    if (i < nsmall) p->gitemsS = uint32_t(gb);
    if (i < nbig) p->gitemsW = uint32_t(gb);
  }
  p->gprefA.push_back(uint32_t(ga));
  p->gitemsA = uint32_t(ga);
  p->gitemsB = uint32_t(gb);
  p->gitemsC = uint32_t(gc);
  p->prefA.push_back(uint32_t(a));
  p->prefB.push_back(uint32_t(b));
  p->prefC.push_back(uint32_t(c));
  p->itemsA = uint32_t(a);
  p->itemsB = uint32_t(b);
  p->itemsC = uint32_t(c);
  p->itemsBb = uint32_t(p->mapBb.size());
  p->itemsBw = uint32_t(p->mapBw.size());
  // a kernel that takes every phase-B item needs no map
  if (p->itemsBb == p->itemsB) p->mapBb.clear();
  if (p->itemsBw == p->itemsB) p->mapBw.clear();
  return NSGC_OK;
}

WsLayout HostPlan::layout() const {
  WsLayout L;
  const size_t e = size_t(ws_elems) * 8;
  size_t o = 0;
  L.keys = o;      o = align_up(o + e, 256);
  L.emit_row = o;  o = align_up(o + e, 256);
  L.emit_col = o;  o = align_up(o + e, 256);
  L.tilemeta = o;  o = align_up(o + size_t(tilemeta_words) * 4, 256);
  L.lbmeta = o;    o = align_up(o + size_t(lbmeta_words) * 4, 256);
  L.rcsize = o;    o = align_up(o + size_t(itemsC) * 4, 256);
  L.order = o;     o = align_up(o + size_t(itemsC) * 4, 256);
  L.partB = o;     o = align_up(o + size_t(itemsB) * 16, 256);
  L.partC = o;     o = align_up(o + size_t(itemsC) * 16, 256);
  if (!gwin.empty()) {
    L.gtile = o;   o = align_up(o + size_t(gtile_words) * 4, 256);
    L.grec = o;    o = align_up(o + size_t(grec_words) * 4, 256);
    L.gheavy = o;  o = align_up(o + gwin.size() * NSGC_GRID_HV_WORDS(NSGC_GRID_HV(gtile_log2)) * 4, 256);
    L.gacc = o;    o = align_up(o + size_t(gitemsB) * 2 * NSGC_GRID_HV(gtile_log2) * 8, 256);
    L.gpartB = o;  o = align_up(o + size_t(gitemsB) * 16, 256);
    L.gpartC = o;  o = align_up(o + size_t(gitemsC) * 16, 256);
    L.goverB = o;  o = align_up(o + size_t(gitemsB) * 4, 256);
    L.goverW = o;  o = align_up(o + size_t(gitemsB) * 4, 256);
    L.goverC = o;  o = align_up(o + size_t(gbuckets) * 8, 256);
  }
  if (num_rows) {
    L.partR = o;   o = align_up(o + size_t(itemsB) * 16, 256);
    L.heavy = o;   o = align_up(o + win.size() * NSGC_HEAVY_SLOTS * 4, 256);
  }
  if (entity) {
    L.partU = o;   o = align_up(o + size_t(itemsC) * 4, 256);
    L.stats = o;   o = align_up(o + tier.size() * 72, 256);
  }
  if (!large.empty()) {   // shared by the large windows, one after another
    L.large = o;   o = align_up(o + large_window_bytes(large_max), 256);
  }
  L.total = std::max<size_t>(o, 256);
  return L;
}

namespace {
struct PlanOffsets {
  size_t small, win, prefA, prefB, prefC, itemwinB, itemwinC, mapBb, mapBw, entcur, entend, gwin,
      gprefA, gitemB, gitemC, total;
};
PlanOffsets plan_offsets(size_t ns, size_t nm, size_t nb, size_t nc, size_t nbb = 0,
                         size_t nbw = 0, size_t nent = 0, size_t ng = 0, size_t ngb = 0,
                         size_t ngc = 0) {
  PlanOffsets o;
  size_t x = align_up(sizeof(nsgc_dev_plan), 64);
  o.small = x; x = align_up(x + ns * sizeof(nsgc_small_desc), 64);
  o.win = x;   x = align_up(x + nm * sizeof(nsgc_win_desc), 64);
  o.prefA = x; x = align_up(x + (nm + 1) * 4, 64);
  o.prefB = x; x = align_up(x + (nm + 1) * 4, 64);
  o.prefC = x; x = align_up(x + (nm + 1) * 4, 64);
  o.itemwinB = x; x = align_up(x + nb * 4, 64);
  o.itemwinC = x; x = align_up(x + nc * 4, 64);
  o.mapBb = x; x = align_up(x + nbb * 4, 64);
  o.mapBw = x; x = align_up(x + nbw * 4, 64);
  o.entcur = x; x = align_up(x + nent * 8, 64);
  o.entend = x; x = align_up(x + nent * 8, 64);
  o.gwin = x;   x = align_up(x + ng * sizeof(nsgc_grid_desc), 64);
  o.gprefA = x; x = align_up(x + (ng + 1) * 4, 64);
  o.gitemB = x; x = align_up(x + ngb * 4, 64);
  o.gitemC = x; x = align_up(x + ngc * 4, 64);
  o.total = x;
  return o;
}
}  // namespace

constexpr size_t kQueueSet = size_t(NSGC_QCLASSES) * NSGC_QSTRIDE * 4;

size_t HostPlan::queue_bytes() const { return (gwin.empty() ? NSGC_Q_GRID : NSGC_Q_ALL) * kQueueSet; }

size_t HostPlan::upload_bytes() const {
  return plan_offsets(small.size(), win.size(), itemwinB.size(), itemwinC.size(), mapBb.size(),
                      mapBw.size(), ent_cur.size(), gwin.size(), gitemB.size(), gitemC.size()).total;
}

namespace {
// Grid windows of a batch of P packets in W windows: by right, and riding along.
void grid_windows_bound(uint64_t P, uint64_t W, uint64_t* gw, uint64_t* riders) {
  *gw = std::min<uint64_t>(W, P / NSGC_GRID_MIN);
  *riders = *gw ? std::min<uint64_t>(std::min<uint64_t>(W, NSGC_GRID_RIDERS), P / NSGC_GRID_RIDE) : 0;
}

// Most cells of `gw` grid windows of P packets in all: a window of n packets
// has fewer than 2 n / target + 2, and at most the cap; one that rides along 16;
// those of a batch below kFinerPackets four times as many.
uint64_t grid_cells_bound(uint64_t P, uint64_t gw, uint64_t riders, const nsgc_tune& t) {
  uint64_t wt = ~uint64_t(0);
  for (int k = 0; k <= 32; ++k)
    if (t.cls[k].wave_target > 0) wt = std::min<uint64_t>(wt, uint64_t(t.cls[k].wave_target));
  if (wt == ~uint64_t(0)) return 0;
  const int cap = std::min(int(t.max_link_buckets_log2), NSGC_GRID_MAX_CELLS_LOG2);
  const uint64_t finer = (uint64_t(1) << kFinerMost) - 1;
  const uint64_t extra = finer * (std::min(P, kFinerPackets) / (2 * wt) +
                                  2 * std::min<uint64_t>(gw, kFinerPackets / NSGC_GRID_MIN));
  return std::min<uint64_t>(P / (2 * wt) + 2 * gw + extra, gw << cap) + riders * 16;
}

// Likewise their phase-C items: R + C < 4 n / target + 4 and at most
// 2^(strips + sub-buckets) each.
uint64_t grid_citems_bound(uint64_t P, uint64_t gw, uint64_t riders, const nsgc_tune& t) {
  uint64_t rt = NSGC_GRID_BUCKET;
  for (int k = 0; k <= 32; ++k)
    rt = std::min<uint64_t>(rt, uint64_t(std::min(t.cls[k].row_target, t.cls[k].col_target)));
  return std::min<uint64_t>(4 * P / rt + 4 * gw,
                            gw * ((uint64_t(1) << (NSGC_GRID_MAX_A + NSGC_GRID_MAX_SUB_LOG2)) +
                                  (uint64_t(1) << (NSGC_GRID_MAX_B + NSGC_GRID_MAX_SUB_LOG2)))) +
         riders * 8 + (gw + riders) * NSGC_GRID_CITEMS(NSGC_GRID_HEAVY);
}
}  // namespace

size_t plan_bound(int64_t max_packets, int64_t max_windows, const nsgc_tune& t) {
  const uint64_t P = uint64_t(std::max<int64_t>(max_packets, 0));
  const uint64_t W = uint64_t(std::max<int64_t>(max_windows, 1));
  uint64_t lt = ~uint64_t(0), rt = ~uint64_t(0);
  for (int k = 0; k <= 32; ++k) {
    lt = std::min<uint64_t>(lt, uint64_t(t.cls[k].link_target));
    rt = std::min<uint64_t>(rt, uint64_t(std::min(t.cls[k].row_target, t.cls[k].col_target)));
  }
  // A bucket count is the power of two at or above ceil(n_w / target) < n_w /
  // target + 1, so B_w < 2 n_w / lt + 2 and R_w + C_w < 4 n_w / rt + 4; each
  // count is also at most its cap (2^max_link_buckets_log2, 2^max_rc_buckets_log2)
  // per window.
  const uint64_t capB = uint64_t(1) << t.max_link_buckets_log2;
  const uint64_t capRC = uint64_t(1) << t.max_rc_buckets_log2;
  const uint64_t nb = std::min<uint64_t>(2 * P / lt + 2 * W, W * capB);
  const uint64_t nc = std::min<uint64_t>(4 * P / rt + 4 * W, 2 * W * capRC);
  // the wavefront buckets (wave_target >= 64) may outnumber the workgroup ones
  uint64_t wt = ~uint64_t(0);
  for (int k = 0; k <= 32; ++k)
    if (t.cls[k].wave_target > 0) wt = std::min<uint64_t>(wt, uint64_t(t.cls[k].wave_target));
  const uint64_t nbw = wt == ~uint64_t(0) ? 0 : std::min<uint64_t>(2 * P / wt + 2 * W, W * capB);
  const uint64_t nb_all = std::max(nb, nbw);
  uint64_t gw, riders;
  grid_windows_bound(P, W, &gw, &riders);
  return plan_offsets(size_t(W), size_t(W), size_t(nb_all), size_t(nc), size_t(nb_all),
                      size_t(nb_all), 0, size_t(gw + riders), size_t(grid_cells_bound(P, gw, riders, t)),
                      size_t(grid_citems_bound(P, gw, riders, t))).total +
         NSGC_Q_ALL * kQueueSet + 1024;
}

size_t grid_workspace_bound(int64_t max_packets, int64_t max_windows, const nsgc_tune& t) {
  const uint64_t P = uint64_t(std::max<int64_t>(max_packets, 0));
  uint64_t gw, riders;
  grid_windows_bound(P, uint64_t(std::max<int64_t>(max_windows, 1)), &gw, &riders);
  if (gw == 0) return 0;
  const uint64_t cells = grid_cells_bound(P, gw, riders, t);
  // tile records: windows of up to 1024 cells in tiles of 2^13 packets (or the
  // tuning's, if smaller; smaller still only below 2 * kGridTiles tiles in all),
  // batches with larger ones in tiles of 2^14
  const uint64_t c13 = std::min<uint64_t>(cells, NSGC_GRID_TILE13_CELLS);
  const uint64_t c14 = std::min<uint64_t>(cells, uint64_t(1) << NSGC_GRID_MAX_CELLS_LOG2);
  const uint64_t t13 = std::max(P >> std::min(t.tile_log2, 13), std::min(P >> 11, 2 * kGridTiles)) + gw + riders;
  const uint64_t tile_words = std::max(t13 * c13, ((P >> 14) + gw + riders) * c14);
  const uint64_t citems = grid_citems_bound(P, gw, riders, t);
  // a cell record has at most 2 NSGC_GRID_MAX_SUB + 3 words, and per window
  // cells * (R / strips + C / strips + 3) <= cells * 3 + (R + C) * max strips
  const uint64_t rec = std::min<uint64_t>(cells * (2 * NSGC_GRID_MAX_SUB + 3),
                                          cells * 3 + (citems << NSGC_GRID_MAX_B));
  return size_t((tile_words + rec + (gw + riders) * NSGC_GRID_HV_WORDS(NSGC_GRID_HEAVY)) * 4 +
                cells * (2 * NSGC_GRID_HEAVY * 8 + 24) + citems * 24 + 9 * 256);
}

void HostPlan::serialize(void* buf, uint64_t dev_plan, uint64_t dev_ws, const uint32_t* src,
                         const uint32_t* dst, void* out) const {
  const PlanOffsets o = plan_offsets(small.size(), win.size(), itemwinB.size(), itemwinC.size(),
                                     mapBb.size(), mapBw.size(), ent_cur.size(), gwin.size(),
                                     gitemB.size(), gitemC.size());
  const WsLayout L = layout();
  char* base = static_cast<char*>(buf);
  std::memset(base, 0, align_up(sizeof(nsgc_dev_plan), 64));
  nsgc_dev_plan h;
  std::memset(&h, 0, sizeof h);
  h.src = src;
  h.dst = dst;
  h.out = static_cast<unsigned long long*>(out);
  h.keys = reinterpret_cast<unsigned long long*>(dev_ws + L.keys);
  h.emit_row = reinterpret_cast<unsigned long long*>(dev_ws + L.emit_row);
  h.emit_col = reinterpret_cast<unsigned long long*>(dev_ws + L.emit_col);
  h.tilemeta = reinterpret_cast<uint32_t*>(dev_ws + L.tilemeta);
  h.lbmeta = reinterpret_cast<uint32_t*>(dev_ws + L.lbmeta);
  h.rcsize = reinterpret_cast<uint32_t*>(dev_ws + L.rcsize);
  h.order = reinterpret_cast<uint32_t*>(dev_ws + L.order);
  h.partB = reinterpret_cast<uint32_t*>(dev_ws + L.partB);
  h.partC = reinterpret_cast<uint32_t*>(dev_ws + L.partC);
  if (num_rows) {
    h.partR = reinterpret_cast<uint32_t*>(dev_ws + L.partR);
    h.heavy = reinterpret_cast<uint32_t*>(dev_ws + L.heavy);
  }
  h.small = reinterpret_cast<const nsgc_small_desc*>(dev_plan + o.small);
  h.win = reinterpret_cast<const nsgc_win_desc*>(dev_plan + o.win);
  h.prefA = reinterpret_cast<const uint32_t*>(dev_plan + o.prefA);
  h.prefB = reinterpret_cast<const uint32_t*>(dev_plan + o.prefB);
  h.prefC = reinterpret_cast<const uint32_t*>(dev_plan + o.prefC);
  h.itemwinB = reinterpret_cast<const uint32_t*>(dev_plan + o.itemwinB);
  h.itemwinC = reinterpret_cast<const uint32_t*>(dev_plan + o.itemwinC);
  h.mapBb = mapBb.empty() ? nullptr : reinterpret_cast<const uint32_t*>(dev_plan + o.mapBb);
  h.mapBw = mapBw.empty() ? nullptr : reinterpret_cast<const uint32_t*>(dev_plan + o.mapBw);
  if (!gwin.empty()) {
    h.gwin = reinterpret_cast<const nsgc_grid_desc*>(dev_plan + o.gwin);
    h.gprefA = reinterpret_cast<const uint32_t*>(dev_plan + o.gprefA);
    h.gitemB = reinterpret_cast<const uint32_t*>(dev_plan + o.gitemB);
    h.gitemC = reinterpret_cast<const uint32_t*>(dev_plan + o.gitemC);
    h.goverB = reinterpret_cast<uint32_t*>(dev_ws + L.goverB);
    h.goverW = reinterpret_cast<uint32_t*>(dev_ws + L.goverW);
    h.goverC = reinterpret_cast<uint32_t*>(dev_ws + L.goverC);
  }
  h.upload16 = uint32_t(upload_bytes() / 16);
  h.clear16 = uint32_t(queue_bytes() / 16);
  h.queue = reinterpret_cast<decltype(h.queue)>(dev_plan + upload_bytes());
  h.num_grid = uint32_t(gwin.size());
  h.gitemsA = gitemsA;
  h.gitemsS = gitemsS;
  h.gitemsW = gitemsW;
  h.gitemsB = gitemsB;
  h.gitemsC = gitemsC;
  h.gtile_log2 = gtile_log2;
  h.itemsBb = itemsBb;
  h.itemsBw = itemsBw;
  h.num_small = entity ? uint32_t(small.size()) : 0u;
  for (int k = 0; k < NSGC_WHOLE; ++k) h.num_whole[k] = num_whole[k];
  h.num_part = uint32_t(win.size());
  h.itemsA = itemsA;
  h.itemsB = itemsB;
  h.itemsC = itemsC;
  h.tile_log2 = tile_log2;
  h.link_slots_log2 = link_slots_log2;
  h.rc_slots_log2 = rc_slots_log2;
  h.small_slots_log2 = small_slots_log2;
  h.max_sweeps_log2 = max_sweeps_log2;
  h.combine_probes = combine_probes;
  h.order_items = itemsC <= NSGC_ORDER_MAX && !entity ? 1u : 0u;
  if (entity) {
    // the statistics go to the workspace; the entity counts to the caller
    h.out = reinterpret_cast<unsigned long long*>(dev_ws + L.stats);
    h.entity = 1;
    h.partU = reinterpret_cast<uint32_t*>(dev_ws + L.partU);
    h.ent_links = static_cast<long long*>(ent_links);
    h.ent_src = static_cast<long long*>(ent_src);
    h.ent_dst = static_cast<long long*>(ent_dst);
    h.ent_counts = static_cast<long long*>(ent_counts);
    h.ent_cur = reinterpret_cast<unsigned long long*>(dev_plan + o.entcur);
    h.ent_end = reinterpret_cast<const unsigned long long*>(dev_plan + o.entend);
  }
  std::memcpy(base, &h, sizeof h);
  if (!small.empty()) std::memcpy(base + o.small, small.data(), small.size() * sizeof(nsgc_small_desc));
  if (!win.empty()) std::memcpy(base + o.win, win.data(), win.size() * sizeof(nsgc_win_desc));
  std::memcpy(base + o.prefA, prefA.data(), prefA.size() * 4);
  std::memcpy(base + o.prefB, prefB.data(), prefB.size() * 4);
  std::memcpy(base + o.prefC, prefC.data(), prefC.size() * 4);
  if (!itemwinB.empty()) std::memcpy(base + o.itemwinB, itemwinB.data(), itemwinB.size() * 4);
  if (!itemwinC.empty()) std::memcpy(base + o.itemwinC, itemwinC.data(), itemwinC.size() * 4);
  if (!mapBb.empty()) std::memcpy(base + o.mapBb, mapBb.data(), mapBb.size() * 4);
  if (!mapBw.empty()) std::memcpy(base + o.mapBw, mapBw.data(), mapBw.size() * 4);
  if (!gwin.empty()) {
    nsgc_grid_desc* gd = reinterpret_cast<nsgc_grid_desc*>(base + o.gwin);
    for (size_t i = 0; i < gwin.size(); ++i) {
      nsgc_grid_desc g = gwin[i];
      g.dst = g.src;
      g.emit_row = g.emit_col = g.keys;
      rebase(g.src, reinterpret_cast<uint64_t>(src));
      rebase(g.dst, reinterpret_cast<uint64_t>(dst));
      rebase(g.keys, dev_ws + L.keys);
      rebase(g.emit_row, dev_ws + L.emit_row);
      rebase(g.emit_col, dev_ws + L.emit_col);
      rebase(g.tile, dev_ws + L.gtile);
      rebase(g.rec, dev_ws + L.grec);
      rebase(g.heavy, dev_ws + L.gheavy);
      rebase(g.acc, dev_ws + L.gacc);
      rebase(g.partB, dev_ws + L.gpartB);
      rebase(g.partC, dev_ws + L.gpartC);
      std::memcpy(gd + i, &g, sizeof g);
    }
    std::memcpy(base + o.gprefA, gprefA.data(), gprefA.size() * 4);
    std::memcpy(base + o.gitemB, gitemB.data(), gitemB.size() * 4);
    std::memcpy(base + o.gitemC, gitemC.data(), gitemC.size() * 4);
  }
  if (!ent_cur.empty()) std::memcpy(base + o.entcur, ent_cur.data(), ent_cur.size() * 8);
  if (!ent_end.empty()) std::memcpy(base + o.entend, ent_end.data(), ent_end.size() * 8);
}

}  // namespace nsgc
