// Short windows: the nine statistics of a window by one workgroup, from the
// packets to the result in one kernel.
//
// The packets stay in registers.  They are inserted in a link table; the
// thread that inserted a link reads its count and adds the link to its source
// in a table of ids, then, in the same memory, to its destination: per link
// and view one insert and one addition, and nothing is scanned, since the
// thread that inserted an id reads its totals.  The tables have twice as many
// slots as the window has packets (one and a half times above 6144), so a short
// window clears few.
//
// Bound by latency: one trip to memory and some ten barriers per window, hidden
// by as many workgroups as fit.  Four sizes: one wavefront, whose barriers cost
// nothing, and 6 KB of LDS for windows of up to 256 packets, of which batches
// have thousands; 4 wavefronts and 25 KB up to 1024; 8 and 49 KB up to 2048; 16
// and 147 KB up to 8192.
// Whole calls, against one kernel with 74 KB of tables for windows of up to
// 1024 packets and the partitioned kernels above (the same plan upload): 2000 windows of 1 .. 1500
// packets 83 -> 45 us, 2000 of 1025 .. 2048 207 -> 67, 500 of 4097 .. 8192 139
// -> 73, one of 8000 47 -> 33; one of 300 the same 16.  One size of 256 threads
// for all windows of up to 1024 packets: 54 us instead of 47 on the first.
#include <hip/hip_runtime.h>

#include "nsgc_device.hpp"
#include "nsgc_grid_device.hpp"
#include "nsgc_phases.hpp"
#include "nsgc_plan.h"
#include "nsgc_whole.hpp"

namespace nsgc {

namespace {

// Source and destination columns, results and windows of a launch.
struct Work {
  const uint32_t* src;
  const uint32_t* dst;
  unsigned long long* out;
  const nsgc_small_desc* list;
};

// `next()` is the workgroup's next window, NO_ITEM at the end, after `ahead()`,
// called once per window a barrier earlier.
template <int NT, int E, int SL, class Next, class Ahead>
__device__ __forceinline__ void whole(const Work& A, uint32_t item, uint32_t* misc, const Next& next,
                                      const Ahead& ahead) {
  constexpr int NW = NT / 64;
  static_assert(SL * 2 >= NT * E * 3, "slots for one and a half times the packets");
  __shared__ __align__(16) u64 tv[SL];        // link keys, then links << 32 | packets of ids
  __shared__ __align__(16) uint32_t tk[SL];   // 16-bit link counts, then ids
  __shared__ uint32_t red[NW][8];
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = lane_id();
  uint16_t* const tc16 = reinterpret_cast<uint16_t*>(tk);
  for (; item != NO_ITEM; item = next()) {
    const nsgc_small_desc D = sload_words(A.list + uniform(item));
    const uint32_t kmax = (D.n + NT - 1) / NT;
    const NSGC_GLOBAL uint32_t* src = gptr(A.src) + D.in_begin;
    const NSGC_GLOBAL uint32_t* dst = gptr(A.dst) + D.in_begin;
    uint32_t r[E], c[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
      r[k] = c[k] = 0;
      if (uint32_t(k) < kmax) {   // (a thread past the end repeats the last packet, masked below)
        const uint32_t i = min(uint32_t(k * NT) + tid, D.n - 1u);
        r[k] = src[i];
        c[k] = dst[i];
      }
    }
    // slots: twice the packets, as far as there are
    const uint32_t S = min(uint32_t(SL), (max(D.n, 32u) * 2u + 63u) & ~63u);
    auto home = [&](uint32_t h) { return __umulhi(h, S); };
    const v4u32 e4 = {EMPTY32, EMPTY32, EMPTY32, EMPTY32}, z4 = {0u, 0u, 0u, 0u};
    for (uint32_t i = tid; i < S / 2; i += NT) reinterpret_cast<v4u32*>(tv)[i] = e4;
    for (uint32_t i = tid; i < S / 8; i += NT) reinterpret_cast<v4u32*>(tk)[i] = z4;
    if (tid < 4) misc[tid] = 0;
    lds_barrier();
    uint32_t at[E];   // slot of a link that this thread inserted
#pragma unroll
    for (int k = 0; k < E; ++k) {
      at[k] = ~0u;
      if (uint32_t(k) < kmax && uint32_t(k * NT) + tid < D.n) {
        r[k] = row_hash(r[k]);
        c[k] = col_hash(c[k]);
        const u64 key = (u64(r[k]) << 32) | c[k];
        if (key == EMPTY64) {   // counted outside the table
          lds_add(&misc[1], 1);
        } else {
          uint32_t s = home(r[k] ^ c[k]);
          for (;;) {   // ends: the table has more slots than the window packets
            const u64 old = lds_cas64(&tv[s], EMPTY64, key);
            if (old == EMPTY64) {
              at[k] = s;
              break;
            }
            if (old == key) {
              lds_add(&tk[s >> 1], 1u << ((s & 1u) << 4));
              break;
            }
            s = s + 1 < S ? s + 1 : 0u;
          }
        }
      }
    }
    lds_barrier();
    uint32_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};   // links, max; ids, max packets, max links per view
    const uint32_t special = misc[1];
#pragma unroll
    for (int k = 0; k < E; ++k)   // from here on `at` is the link's packets, 0 for none
      if (uint32_t(k) < kmax) {
        at[k] = at[k] != ~0u ? tc16[at[k]] + 1u : 0u;
        v[0] += at[k] ? 1u : 0u;
        v[1] = max(v[1], at[k]);
      }
    if (tid == 0 && special) {
      ++v[0];
      v[1] = max(v[1], special);
    }
#pragma unroll
    for (int view = 0; view < 2; ++view) {
      lds_barrier();
      for (uint32_t i = tid; i < S / 2; i += NT) reinterpret_cast<v4u32*>(tv)[i] = z4;
      for (uint32_t i = tid; i < S / 4; i += NT) reinterpret_cast<v4u32*>(tk)[i] = e4;
      if (tid == 2) misc[2] = special;
      if (tid == 3) misc[3] = special ? 1u : 0u;
      lds_barrier();
      uint32_t own[E];
#pragma unroll
      for (int k = 0; k < E; ++k) {
        own[k] = ~0u;
        if (uint32_t(k) < kmax && at[k]) {
          const uint32_t id = view ? c[k] : r[k];
          if (id == EMPTY32) {   // the hashed id EMPTY32 lives outside the table
            lds_add(&misc[2], at[k]);
            lds_add(&misc[3], 1);
          } else {
            uint32_t s = home(id);
            for (;;) {
              const uint32_t old = lds_cas32(&tk[s], EMPTY32, id);
              if (old == EMPTY32) own[k] = s;
              if (old == EMPTY32 || old == id) break;
              s = s + 1 < S ? s + 1 : 0u;
            }
            lds_add64(&tv[s], (u64(1) << 32) | at[k]);
          }
        }
      }
      lds_barrier();
#pragma unroll
      for (int k = 0; k < E; ++k)
        if (uint32_t(k) < kmax && own[k] != ~0u) {
          const u64 x = tv[own[k]];
          ++v[2 + 3 * view];
          v[3 + 3 * view] = max(v[3 + 3 * view], uint32_t(x));
          v[4 + 3 * view] = max(v[4 + 3 * view], uint32_t(x >> 32));
        }
      if (tid == 0 && misc[3]) {
        ++v[2 + 3 * view];
        v[3 + 3 * view] = max(v[3 + 3 * view], misc[2]);
        v[4 + 3 * view] = max(v[4 + 3 * view], misc[3]);
      }
    }
    ahead();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool sum = k == 0 || k == 2 || k == 5;
      v[k] = sum ? wave_sum(v[k]) : wave_max(v[k]);
      if (lane == 0) red[w][k] = v[k];
    }
    lds_barrier();
    if (tid < 9) {   // the packets, then v in its order
      uint32_t x = D.n;
      if (tid) {
        const bool sum = tid == 1 || tid == 3 || tid == 6;
        x = 0;
        for (int k = 0; k < NW; ++k) x = sum ? x + red[k][tid - 1] : max(x, red[k][tid - 1]);
      }
      gptr(A.out)[u64(D.out_index) * 9 + tid] = x;
    }
    lds_barrier();
  }
}

// The windows of an uploaded plan, from its list.
template <int NT, int E, int SL>
__global__ __launch_bounds__(NT) void k_whole(nsgc_dev_plan* P, uint32_t which) {
  __shared__ uint32_t misc[8];   // 1 special packets, 2 / 3 special id's packets / links, 7 queue slot
  const uint32_t items = sload(&P->num_whole[which]);
  uint32_t first = 0;
  for (uint32_t k = 0; k < which; ++k) first += sload(&P->num_whole[k]);
  const Work A = {sload(&P->src), sload(&P->dst), sload(&P->out), sload(&P->small) + first};
  ItemQueue q(gptr(&sload(&P->queue)[NSGC_Q_WHOLE + which][0]), misc + 7, NSGC_QCLASSES);
  whole<NT, E, SL>(A, q.first(items), misc, [&]() { return q.read(); }, [&]() { q.stage_next(items); });
}

// A few windows without a plan: they come with the launch, a workgroup each.
constexpr int FEW = 224;
struct FewWindows {
  Work A;
  nsgc_small_desc list[FEW];
};
static_assert(sizeof(FewWindows) <= 3968, "kernel arguments");

template <int NT, int E, int SL>
__global__ __launch_bounds__(NT) void k_whole_few(FewWindows) {
  __shared__ uint32_t misc[8];
  // (the arguments where they lie: indexed, they would be copied first)
  const FewWindows* args = (const FewWindows*)__builtin_amdgcn_kernarg_segment_ptr();
  const Work A = {sload(&args->A.src), sload(&args->A.dst), sload(&args->A.out), args->list};
  whole<NT, E, SL>(A, blockIdx.x, misc, []() { return NO_ITEM; }, []() {});
}

void (*const whole_kernels[NSGC_WHOLE])(nsgc_dev_plan*, uint32_t) = {
    &k_whole<NSGC_WHOLE_A / 4, 4, 2 * NSGC_WHOLE_A>,
    &k_whole<NSGC_WHOLE_B / 4, 4, 2 * NSGC_WHOLE_B>,
    &k_whole<NSGC_WHOLE_C / 4, 4, 2 * NSGC_WHOLE_C>,
    &k_whole<NSGC_WHOLE_D / 8, 8, 3 * NSGC_WHOLE_D / 2>,
};
void (*const few_kernels[NSGC_WHOLE])(FewWindows) = {
    &k_whole_few<NSGC_WHOLE_A / 4, 4, 2 * NSGC_WHOLE_A>,
    &k_whole_few<NSGC_WHOLE_B / 4, 4, 2 * NSGC_WHOLE_B>,
    &k_whole_few<NSGC_WHOLE_C / 4, 4, 2 * NSGC_WHOLE_C>,
    &k_whole_few<NSGC_WHOLE_D / 8, 8, 3 * NSGC_WHOLE_D / 2>,
};
const int whole_threads[NSGC_WHOLE] = {NSGC_WHOLE_A / 4, NSGC_WHOLE_B / 4, NSGC_WHOLE_C / 4, NSGC_WHOLE_D / 8};

}  // namespace

hipError_t launch_whole(const nsgc_dev_plan* P, int which, uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(whole_kernels[which], dim3(grid), dim3(whole_threads[which]), 0, s,
                     const_cast<nsgc_dev_plan*>(P), uint32_t(which));
  return hipGetLastError();
}

bool whole_few(size_t windows) { return windows > 0 && windows <= size_t(FEW); }

hipError_t launch_whole_few(int which, const nsgc_small_desc* list, size_t windows, const uint32_t* src,
                            const uint32_t* dst, void* out, hipStream_t s) {
  FewWindows f;
  f.A = {src, dst, static_cast<unsigned long long*>(out), nullptr};
  for (size_t i = 0; i < windows; ++i) f.list[i] = list[i];
  hipLaunchKernelGGL(few_kernels[which], dim3(uint32_t(windows)), dim3(whole_threads[which]), 0, s, f);
  return hipGetLastError();
}

hipError_t whole_resident_blocks(int which, int* blocks) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(
      blocks, reinterpret_cast<const void*>(whole_kernels[which]), whole_threads[which], 0);
}

}  // namespace nsgc
