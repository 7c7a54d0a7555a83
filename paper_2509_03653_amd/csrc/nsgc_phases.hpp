// Shared by the phase-B and phase-C kernels: the emission entries and the walk
// over an item's segments.
#ifndef NSGC_PHASES_HPP_
#define NSGC_PHASES_HPP_

#include <type_traits>

#include "nsgc_device.hpp"

namespace nsgc {

template <class A>
__host__ __device__ constexpr int array_len() {
  return int(std::extent<std::remove_reference_t<A>>::value);
}

// Probes before an insert of phases B and C gives up; the caller then splits
// the keys into sweeps, so giving up never changes a result.
constexpr uint32_t NSGC_MAX_PROBES = 64;

// The tables of the grid's phases and of the entity outputs are probed in steps
// of an odd number that the key decides, from bits that neither its bucket nor its
// home slot takes.  (Consecutive slots would form chains: a table of 4096 slots
// has one of more than 64 from three fifths full on, against nine tenths.)
__device__ __forceinline__ uint32_t probe_step(u64 link) { return (uint32_t(link >> 45) ^ (uint32_t(link) >> 13)) | 1u; }
__device__ __forceinline__ uint32_t probe_step(uint32_t id) { return (id >> 12) | 1u; }

// Second half of a find-or-insert of one key per lane in an open-addressing
// LDS table: `old` is what the compare-and-swap on the home slot returned, `slot`
// goes in as the home slot and out as the slot last tried.  Returns what that
// slot held: the table's marker if the key was inserted, the key if it was there,
// anything else if it found no place within `most` probes.
// (Plain values, no flags: flags carried through a divergent loop cost scalar
// instructions per step.)
template <class K>
__device__ __forceinline__ K probe_on(K* tk, uint32_t mask, K key, K old, uint32_t& slot,
                                      uint32_t most = NSGC_MAX_PROBES) {
  constexpr K EMPTY = K(~K(0));
  for (uint32_t left = most - 1; old != EMPTY && old != key && left; --left) {
    slot = (slot + probe_step(key)) & mask;
    if constexpr (sizeof(K) == 8) old = lds_cas64(reinterpret_cast<u64*>(tk) + slot, EMPTY64, key);
    else old = lds_cas32(reinterpret_cast<uint32_t*>(tk) + slot, EMPTY32, key);
  }
  return old;
}
constexpr uint32_t ENT_PMAX = (1u << NSGC_ENT_PACKET_BITS) - 1;
constexpr uint32_t ENT_LMAX = (1u << NSGC_ENT_LINK_BITS) - 1;
static_assert(NSGC_ENT_PACKET_BITS + NSGC_ENT_LINK_BITS == 32, "entry fields");

// Entries needed for an (id, links, packets) triple (1 <= links <= packets).
__device__ __forceinline__ uint32_t entry_parts(uint32_t packets, uint32_t links) {
  if (packets <= ENT_PMAX && links <= ENT_LMAX) return 1u;
  const uint32_t a = packets / ENT_PMAX + (packets % ENT_PMAX != 0);
  const uint32_t b = links / ENT_LMAX + (links % ENT_LMAX != 0);
  return max(max(a, b), 1u);
}

// Write the `parts` entries of a triple at e[at], e[at + 1], ...
__device__ __forceinline__ void write_entry(NSGC_GLOBAL u64* e, uint32_t at, uint32_t id,
                                            uint32_t packets, uint32_t links, uint32_t parts) {
  if (parts == 1) {
    e[at] = (u64(id) << 32) | (u64(links) << NSGC_ENT_PACKET_BITS) | packets;
    return;
  }
  const uint32_t pq = packets / parts, pr = packets % parts;
  const uint32_t lq = links / parts, lr = links % parts;
  for (uint32_t i = 0; i < parts; ++i) {
    const uint32_t p = pq + (i < pr), l = lq + (i < lr);
    e[at + i] = (u64(id) << 32) | (u64(l) << NSGC_ENT_PACKET_BITS) | p;
  }
}

// ---------------------------------------------------------------------------
// Shared machinery of phases B and C: visit the elements of `nseg` segments
// (`seg(i, base, len)` describes segment i) wavefront by wavefront.
//
// Wavefront w of NW takes segments w, w + NW, w + 2 NW, ... of each group of
// 64 * NW segments; its lanes load the descriptions of the wave's (up to
// 64) segments at once, and the wave walks them in chunks of 64 consecutive
// elements, up to MAXU chunks per round.  Long segments are walked one at a
// time (lane = offset in the chunk; a segment's last chunk may be partly
// idle).  When the segments are short (large windows cut into many buckets
// and tiles) that would leave most lanes idle, so the wave instead walks the
// concatenation of its segments: lane l of a chunk at position v takes
// element v + l, whose segment a 6-step binary search over the lanes'
// inclusive length prefix finds.  There is no LDS staging and no barrier
// until the one at the end, so waves proceed independently.  `fn(pos, ok)`
// receives the round's positions (pos[u] valid when ok[u]; the array length
// is the round's unroll) with the whole wavefront active; it must not use
// workgroup barriers.
// ---------------------------------------------------------------------------

__device__ __forceinline__ u64 readlane64(u64 v, uint32_t k) {
  return (u64(readlane(uint32_t(v >> 32), int(k))) << 32) | readlane(uint32_t(v), int(k));
}

// Rounds over `total` chunks (uniform across the wavefront, not the block):
// body(integral_constant<int, UU>) with the smallest UU of 8, 4, 2, 1 (at
// most MAXU) that covers what is left.
template <int MAXU, class Body>
__device__ __forceinline__ void for_chunk_rounds(uint32_t total, Body&& body) {
  static_assert(MAXU == 8 || MAXU == 4 || MAXU == 2 || MAXU == 1, "unroll");
  for (uint32_t c = 0; c < total;) {
    const uint32_t rem = total - c;
    if (MAXU >= 8 && rem > 4) {
      body(std::integral_constant<int, (MAXU >= 8 ? 8 : 1)>());
      c += 8;
    } else if (MAXU >= 4 && rem > 2) {
      body(std::integral_constant<int, (MAXU >= 4 ? 4 : 1)>());
      c += 4;
    } else if (MAXU >= 2 && rem > 1) {
      body(std::integral_constant<int, (MAXU >= 2 ? 2 : 1)>());
      c += 2;
    } else {
      body(std::integral_constant<int, 1>());
      c += 1;
    }
  }
}

// Keeps a wave-uniform value in a scalar register (the compiler cannot always
// prove uniformity of values derived from threadIdx.x / 64).
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
  return uint32_t(__builtin_amdgcn_readfirstlane(int(v)));
}

// The packed walk is taken when it needs fewer than PACK_NUM / PACK_DEN of
// the segment-by-segment walk's chunks (its search costs part of a chunk).
constexpr uint32_t PACK_NUM = 7, PACK_DEN = 8;

// This lane's segment of the first group (segments w + WAVES * lane), when
// the caller loaded it beforehand (zero length where there is none).
struct SegPre {
  u64 base;
  uint32_t len;
};

struct NoTail {
  __device__ void operator()() const {}
};

// `tail()` runs in every thread just before the final barrier.
template <int MAXU, int NW = WAVES, class SegFn, class BatchFn, class Tail = NoTail>
__device__ __forceinline__ void gather_by_wave(uint32_t nseg, SegFn seg, BatchFn fn,
                                               const SegPre* pre = nullptr, Tail tail = Tail()) {
  const uint32_t w = uniform(threadIdx.x >> 6), lane = lane_id();
  constexpr uint32_t GROUP = 64u * uint32_t(NW);
  constexpr int PACKU = MAXU < 4 ? MAXU : 4;
  for (uint32_t g0 = 0; g0 < nseg; g0 += GROUP) {
    const uint32_t si = g0 + w + uint32_t(NW) * lane;   // this lane's segment
    u64 mybase = 0;
    uint32_t mylen = 0;
    if (g0 == 0 && pre) {
      mybase = pre->base;
      mylen = pre->len;
    } else if (si < nseg) {
      seg(si, mybase, mylen);
    }
    const uint32_t nk = uniform(g0 + w < nseg ? min(64u, (nseg - g0 - w + NW - 1) / NW) : 0u);
    const uint32_t chunks = uniform(wave_sum((mylen + 63u) >> 6));   // segment by segment
    const uint32_t elems = uniform(wave_sum(mylen));
    const uint32_t packed_chunks = (elems + 63u) >> 6;               // concatenated
    if (PACK_DEN * packed_chunks < PACK_NUM * chunks) {
      // Packed walk, in rounds of at most 4 chunks (the search's registers
      // stay out of the widest round).  Lane l of the chunk at v takes
      // element v + l of the concatenation; its segment j is the number of
      // lanes whose inclusive prefix is <= v + l (empty segments skipped).
      const uint32_t incl = wave_inclusive_scan(mylen);
      const u64 mb = mybase - (incl - mylen);   // base - exclusive prefix
      uint32_t v0 = 0;
      for_chunk_rounds<PACKU>(packed_chunks, [&](auto uc) {
        constexpr int U = decltype(uc)::value;
        u64 pos[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t v = v0 + lane;
          uint32_t j = 0;
#pragma unroll
          for (uint32_t st = 32; st > 0; st >>= 1)
            if (lane_take(incl, j + st - 1) <= v) j += st;
          pos[u] = ((u64(lane_take(uint32_t(mb >> 32), j)) << 32) | lane_take(uint32_t(mb), j)) + v;
          ok[u] = v < elems;
          v0 = uniform(v0 + 64);
        }
        fn(pos, ok);
      });
      continue;
    }
    uint32_t k = 0, off = 0;                                          // uniform cursor
    while (k < nk && readlane(mylen, int(k)) == 0) k = uniform(k + 1);
    for_chunk_rounds<MAXU>(chunks, [&](auto uc) {
      constexpr int U = decltype(uc)::value;
      u64 pos[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (k < nk) {
          const uint32_t len = readlane(mylen, int(k));
          pos[u] = readlane64(mybase, k) + off + lane;
          ok[u] = off + lane < len;
          off = uniform(off + 64);
          if (off >= len) {
            off = 0;
            k = uniform(k + 1);
            while (k < nk && readlane(mylen, int(k)) == 0) k = uniform(k + 1);
          }
        } else {
          pos[u] = 0;
          ok[u] = false;
        }
      }
      fn(pos, ok);
    });
  }
  tail();
  __syncthreads();
}

}  // namespace nsgc

#endif  // NSGC_PHASES_HPP_
