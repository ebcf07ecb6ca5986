// Device-side building blocks shared by the reconstruction and distance
// transform kernels (gfx950, wave64).
//
// Cross-workgroup coherence.  On MI355X every XCD has its own L2 and the L2s
// are not coherent with each other while a kernel runs, so plain loads can
// return stale lines for data another XCD wrote during the same launch.  The
// persistent kernels therefore move all data that other workgroups of the same
// launch read or write with device-scope ("sc1") loads and stores, and publish
// it by draining the store counter (s_waitcnt vmcnt(0)) before the atomic
// that makes it reachable.  The alternative -- agent-scope acquire/release,
// which writes back and invalidates the whole L2 -- costs roughly ten times
// more per handoff.  Kernel boundaries are coherence points, so data written
// by an earlier kernel may be read with plain loads.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "iwpp_barrier.hpp"

namespace iwpp {

constexpr int kWave = 64;
constexpr int kSc1 = 16;  // buffer-instruction cache policy bit: device scope

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, 0x00020000);
}

// Wait until every store/atomic this wave issued has completed.
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---- device-coherent scalar accesses (one element per lane) -----------------
template <typename T>
__device__ __forceinline__ T cload(const T* p) {
  return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void cstore(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T atomic_add(T* p, T v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T atomic_or(T* p, T v) {
  return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T atomic_max(T* p, T v) {
  return __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- wave helpers -------------------------------------------------------------
__device__ __forceinline__ int lane() { return (int)__lane_id(); }
// A per-lane value the compiler knows nothing about: what is computed from it
// is computed where it is used.  In a persistent kernel it would otherwise be
// moved out of all loops, kept in registers over the whole kernel and, past
// their number, in scratch memory, whose reloads wait behind a visit's stores.
__device__ __forceinline__ int local_copy(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
// The kernel's only argument, read again from where it lies (scalar loads).  In
// a persistent kernel the fields would otherwise be read once, kept in scalar
// registers over all loops and, past their number, in lanes of vector registers,
// sixteen of them brought back for one that is needed (16384^2 reconstruction
// 1507 us, read again in each visit 1487).
template <typename Args>
__device__ __forceinline__ Args kernel_args() {
  static_assert(sizeof(Args) % 8 == 0, "read by 8-byte words");
  typedef const __attribute__((address_space(4))) uint64_t* Words;
  Words p = (Words)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  struct Raw {
    uint64_t w[sizeof(Args) / 8];
  } r;
#pragma unroll
  for (size_t k = 0; k < sizeof(Args) / 8; ++k) r.w[k] = p[k];
  return __builtin_bit_cast(Args, r);
}
__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
__device__ __forceinline__ int mbcnt(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// lane i receives v from lane i-1; lane 0 receives `fill`.
__device__ __forceinline__ uint32_t from_left(uint32_t v, uint32_t fill) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)fill, (int)v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}
// lane i receives v from lane i+1; lane 63 receives `fill`.
__device__ __forceinline__ uint32_t from_right(uint32_t v, uint32_t fill) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)fill, (int)v, 0x130 /* wave_shl:1 */, 0xf, 0xf, false);
}
// A value the wave holds in common, moved to scalar registers word by word
// (e.g. a job descriptor read through a per-tile table), so that buffer
// resources built from it need no per-lane loop.
template <class V>
__device__ __forceinline__ V uniform(const V& v) {
  static_assert(sizeof(V) % 4 == 0, "whole words");
  uint32_t w[sizeof(V) / 4];
  __builtin_memcpy(w, &v, sizeof(V));
#pragma unroll
  for (int i = 0; i < (int)(sizeof(V) / 4); ++i) w[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[i]);
  V r;
  __builtin_memcpy(&r, w, sizeof(V));
  return r;
}
// Inclusive prefix sum over the 64 lanes with DPP (no LDS round trips):
// shifts by 1, 2, 4 and 8 inside each row of 16 lanes (zero-filled), then row
// 0's total into row 1 and row 2's into row 3 (row_bcast:15), then the total of
// rows 0-1 into rows 2-3 (row_bcast:31).
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111 /* row_shr:1 */, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112 /* row_shr:2 */, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114 /* row_shr:4 */, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118 /* row_shr:8 */, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142 /* row_bcast:15 */, 0xa, 0xf, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143 /* row_bcast:31 */, 0xc, 0xf, false);
  return x;
}
__device__ __forceinline__ uint32_t readlane(uint32_t v, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

// ---- statistics: sharded counters (8 copies, one per workgroup group) ---------
// Fields are summed over the shards by the host.
enum StatField : int {
  kStatSeeds = 0,
  kStatItems = 1,
  kStatSweeps = 2,
  kStatRounds = 3,
  kStatUpdates = 4,
  kStatRestarts = 5,
  kStatError = 6,
  kStatFields = 16
};
constexpr int kStatShards = 8;

__device__ __forceinline__ void stat_add(unsigned long long* stats, int field, unsigned long long v) {
  if (v) atomic_add(stats + (blockIdx.x & (kStatShards - 1)) * kStatFields + field, v);
}

// ---- grid barrier ---------------------------------------------------------------
// Counting barrier for a co-resident (cooperative) grid (state and protocol:
// iwpp_barrier.hpp).  A workgroup counts itself in one of 8 group counters
// (blockIdx & 7), the last of a group writes the group's word of this generation,
// and everyone polls the eight words -- half a cache line -- with the abort word in
// the same load.  Every wait is bounded: on timeout (or when another workgroup
// raised `abort`) the barrier returns false and the caller must leave the kernel.
//
// A round with few tiles is mostly latencies, so the barrier has two memory
// round trips on its path.  Counters only grow: nothing is reset, and nothing has
// to be written before the generation.  Before, with a counter over the groups,
// resets, and generation, abort word and result read one after the other, a
// 389 x 517 transform (12 steps) took 325 us, now 309; a 4096^2 reconstruction 340
// and 331, 32 small images 1195 and 1164.
//
// The items appended travel with the arrivals, so that a round begins with its
// lists' lengths known and no more loads.  With it, and with shares cut without
// 64-bit divisions and items read from the group's own sub-list without a search,
// a reconstruction of 512 x 512 went from 143 to 120 us, 1500 x 1301 187 to 165,
// 4096^2 307 to 282, 65536 x 65600 15990 to 14730.
constexpr uint32_t kSpinLimit = 1u << 24;  // ~ seconds of polling, far beyond any real wait

// What the kernel's workgroup has appended since the last barrier (LDS), and
// the items of each group up to then (lane x of wave 0: group x).
struct Appended {
  uint32_t* here;
  uint32_t* cnt;  // LDS: per group, filled by the barrier with what the grid appended since the last
  uint32_t* zero;  // LDS word the barrier clears (null: none)
  uint32_t seen;
};

// Every wave first waits for its own stores: none is in flight when the
// workgroup is counted.
__device__ __forceinline__ bool grid_barrier(GridBarrier* b, uint32_t& gen, unsigned long long* stats,
                                             Appended* app = nullptr) {
  __shared__ uint32_t ok;
  drain();
  __syncthreads();
  if (threadIdx.x < (unsigned)kWave) {  // wave 0
    const uint32_t nwg = gridDim.x, g = blockIdx.x & 7u, in_group = (nwg - g + 7u) >> 3, groups = nwg < 8u ? nwg : 8u;
    const uint32_t l = (uint32_t)local_copy((int)threadIdx.x);
    unsigned long long* words = b->word[barrier::slot(gen)];
    if (l == 0u) {
      const unsigned long long one = barrier::arrival(app ? *app->here : 0u);
      const unsigned long long total = atomic_add(&b->group[g][0], one) + one;
      if (barrier::last(total, gen, in_group)) cstore(&words[g], barrier::word(total, gen));
      if (app) {
        *app->here = 0u;
        if (app->zero) *app->zero = 0u;
      }
    }
    unsigned long long v = 0ull;
    uint32_t res = 1;
    for (uint32_t spins = 0;;) {
      uint32_t stop = 0u;
      if (l < groups) v = cload(&words[l]);
      if (l == groups) stop = cload(&b->abort[0]);
      if (ballot(stop != 0u) != 0ull) {
        res = 0;
        break;
      }
      if (ballot(l < groups && !barrier::arrived(v, gen)) == 0ull) break;
      __builtin_amdgcn_s_sleep(2);
      if (++spins > kSpinLimit) {
        if (l == 0u) {
          cstore(&b->abort[0], 1u);
          atomic_add(stats + kStatError, 1ull);
        }
        res = 0;
        break;
      }
    }
    if (app && l < 8u) {
      const uint32_t items = barrier::items(v);
      app->cnt[l] = items - app->seen;
      app->seen = items;
    }
    if (l == 0u) ok = res;
  }
  __syncthreads();
  gen += 1u;
  return ok != 0;
}

// Compiler + memory ordering point for lanes of one wave that exchange data
// through LDS (LDS instructions of a wave execute in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---- per-wave staged append ---------------------------------------------------
// A wave collects items in an LDS buffer with ballot + mbcnt (no atomics) and
// flushes it to a global list with one atomic per flush.  `cap_global` bounds
// the global list; items past it are dropped and *ovf is set.  The fill level
// `n` is wave-uniform and lives in a register.
template <typename Item>
struct WaveStageT {
  Item* items;  // LDS, `cap` entries
  uint32_t cap;
  uint32_t n;
};
using WaveStage = WaveStageT<uint32_t>;

template <typename Item>
__device__ __forceinline__ void stage_flush(WaveStageT<Item>& s, Item* list, uint32_t* count, uint32_t cap_global,
                                            uint32_t* ovf) {
  const uint32_t n = s.n;
  if (n == 0) return;
  wave_sync();
  uint32_t base = 0;
  if (lane() == 0) base = atomic_add(count, n);
  base = readlane(base, 0);
  for (uint32_t i = lane(); i < n; i += kWave) {
    uint32_t slot = base + i;
    if (slot < cap_global) cstore(list + slot, s.items[i]);
  }
  if (base + n > cap_global && lane() == 0) cstore(ovf, 1u);
  wave_sync();
  s.n = 0;
}

// Append `item` for every lane with `pred`; flushes first if the stage could overflow.
template <typename Item>
__device__ __forceinline__ void stage_append(WaveStageT<Item>& s, bool pred, Item item, Item* list, uint32_t* count,
                                             uint32_t cap_global, uint32_t* ovf) {
  const uint64_t m = ballot(pred);
  if (m == 0) return;
  const uint32_t k = (uint32_t)__popcll(m);
  if (s.n + k > s.cap) stage_flush(s, list, count, cap_global, ovf);
  if (pred) s.items[s.n + mbcnt(m)] = item;
  s.n += k;
}

// ---- round timeline -----------------------------------------------------------
// Workgroup 0 stamps the realtime clock (a constant-rate counter) at kernel
// start and after every grid barrier into words 1..255 (word 0 counts the
// stamps), and the work of each phase (tiles visited) into words 256 + phase.
// Costs one or two stores per round.
constexpr uint32_t kClockStamps = 256;
__device__ __forceinline__ void clock_stamp(unsigned long long* clock, uint32_t& n) {
  if (blockIdx.x == 0 && threadIdx.x == 0 && n + 1u < kClockStamps) {
    n++;
    clock[n] = __builtin_amdgcn_s_memrealtime();
    clock[0] = n;
  }
}
__device__ __forceinline__ void round_work(unsigned long long* clock, uint32_t phase, uint32_t tiles) {
  if (blockIdx.x == 0 && threadIdx.x == 0 && phase < kClockStamps) clock[kClockStamps + phase] = tiles;
}

// Work of a round shared by the waves of a workgroup: the workgroup owns a
// contiguous range [lo, hi) of the round's items, and its waves take the next
// item from an LDS counter, so a wave whose visits were cheap takes more.
// Ranges are cut XCD-major: workgroup b runs on XCD b mod 8, and the eight
// XCDs own eight contiguous parts of the items, so the tiles an XCD visits
// together are neighbours whose shared cache lines (the other half of a
// 128-byte line, the halo rows and border columns) its own L2 holds.
// (One device-scope atomic per item instead, shared by all workgroups, was
// measured to double the dense rounds: its latency under contention exceeds
// the imbalance it removes; items dealt round-robin over the workgroups made
// the seed pass 40% slower than neighbouring strips on one XCD.)
struct WgShare {
  uint32_t lo, hi;
  uint32_t* next;  // LDS, zeroed before the round
  __device__ bool take(uint32_t& i) const {
    uint32_t k = 0;
    if (lane() == 0) k = atomicAdd(next, 1u);
    k = readlane(k, 0);
    i = lo + k;
    return i < hi;
  }
};

constexpr uint32_t kXcds = 8;  // workgroup b runs on XCD b mod 8

// Workgroups of the grid on XCD x, and this workgroup's rank among them.
__device__ __forceinline__ uint32_t xcd_groups(uint32_t x) { return (gridDim.x + kXcds - 1u - x) / kXcds; }

// First item of part l of n items cut into L parts whose sizes differ by one at most.
__device__ __forceinline__ uint32_t part_begin(uint32_t n, uint32_t l, uint32_t L) {
  const uint32_t q = n / L, r = n - q * L;
  return q * l + (l < r ? l : r);
}

// This workgroup's share of the items [base, base + n) owned by its XCD.
__device__ __forceinline__ WgShare share_of(uint32_t base, uint32_t n, uint32_t* next) {
  const uint32_t l = blockIdx.x / kXcds, L = xcd_groups(blockIdx.x % kXcds);
  WgShare w;
  w.lo = base + part_begin(n, l, L);
  w.hi = base + part_begin(n, l + 1u, L);
  w.next = next;
  return w;
}

// n items cut into eight XCD parts (when the grid covers all XCDs).
__device__ __forceinline__ WgShare wg_share(uint32_t n, uint32_t* next) {
  if (gridDim.x < kXcds) {
    WgShare w;
    w.lo = part_begin(n, blockIdx.x, gridDim.x);
    w.hi = part_begin(n, blockIdx.x + 1u, gridDim.x);
    w.next = next;
    return w;
  }
  const uint32_t x = blockIdx.x % kXcds;
  const uint32_t lo = part_begin(n, x, kXcds), hi = part_begin(n, x + 1u, kXcds);
  return share_of(lo, hi - lo, next);
}

// ---- sharded tile frontier --------------------------------------------------------
// A round's work list of tiles is split into kShards sub-lists, one per group of
// workgroups (blockIdx & 7, i.e. one per XCD).  A wave stages its appends in LDS
// and flushes them into its group's sub-list with one atomic on that sub-list's
// counter, so each counter sees an eighth of the flushes.  In the next round a
// group consumes its own sub-list, whose tiles are neighbours of those it visited
// last.  A per-tile flag word (set with atomic_or) keeps a tile on a round's list
// at most once.
constexpr int kShards = 8;

// Counter of (round slot, shard): 256 bytes apart.
__device__ __forceinline__ uint32_t* shard_count(uint32_t* counts, uint32_t slot, uint32_t shard) {
  return counts + (slot * (uint32_t)kShards + shard) * 64u;
}

// Flush the stage into sub-list `list` (capacity `cap`) counted by `count`.
// Items past the capacity are dropped: their flag is cleared (so a later mark
// can list them again) and *lost is set.
__device__ inline void shard_flush(WaveStage& s, uint32_t* list, uint32_t* count, uint32_t cap, uint32_t* flags,
                                   uint32_t* lost, uint32_t* appended) {
  const uint32_t n = s.n;
  if (n == 0) return;
  wave_sync();
  const uint32_t l = (uint32_t)local_copy(lane());
  uint32_t base = 0;
  if (l == 0u) {
    base = atomic_add(count, n);
    atomicAdd(appended, n);  // LDS: the workgroup's, for the barrier
  }
  base = readlane(base, 0);
  bool dropped = false;
  for (uint32_t i = l; i < n; i += kWave) {
    const uint32_t slot = base + i, item = s.items[i];
    if (slot < cap) {
      cstore(list + slot, item);
    } else {
      cstore(flags + item, 0u);
      dropped = true;
    }
  }
  if (ballot(dropped) && l == 0u) cstore(lost, 1u);
  wave_sync();
  s.n = 0;
}

// Stage tile t (every lane with `pred`) unless it is already on the list
// whose flags are `flags`; flushes first if the stage could overflow.
__device__ inline void shard_mark(WaveStage& s, bool pred, uint32_t t, uint32_t* flags, uint32_t* list,
                                  uint32_t* count, uint32_t cap, uint32_t* lost, uint32_t* appended) {
  const bool fresh = pred && atomic_or(flags + t, 1u) == 0u;
  const uint64_t m = ballot(fresh);
  if (m == 0) return;
  const uint32_t k = (uint32_t)__popcll(m);
  if (s.n + k > s.cap) shard_flush(s, list, count, cap, flags, lost, appended);
  if (fresh) s.items[s.n + mbcnt(m)] = t;
  s.n += k;
}

// Length of round slot `slot`'s list: per-shard counts (capped) into `cnt`
// (kShards entries in LDS, filled by threads 0..kShards-1 of the workgroup).
__device__ __forceinline__ void shard_counts(uint32_t* counts, uint32_t slot, uint32_t cap, uint32_t* cnt) {
  if (threadIdx.x < (unsigned)kShards) {
    const uint32_t c = cload(shard_count(counts, slot, threadIdx.x));
    cnt[threadIdx.x] = c < cap ? c : cap;
  }
}

// Item i of the concatenated sub-lists of one parity (lists: [kShards][stride]).
__device__ __forceinline__ uint32_t shard_item(const uint32_t* lists, uint32_t stride, const uint32_t* cnt, uint32_t i) {
  uint32_t x = 0;
  while (x + 1 < (uint32_t)kShards && i >= cnt[x]) {
    i -= cnt[x];
    ++x;
  }
  return cload(lists + (size_t)x * stride + i);
}

}  // namespace iwpp
