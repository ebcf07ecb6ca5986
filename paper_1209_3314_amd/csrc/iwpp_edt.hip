// Propagation-based Euclidean distance transform on gfx950.
//
// What is computed (Sec. 2.2, Algorithms 3 and 6): every pixel carries a
// nearest feature (the paper's VR), initially itself for features (0-pixels)
// and "none" otherwise; features propagate to neighbours in N_G when they are
// closer; the output is the squared distance to the carried feature and its
// index.  The propagation runs in level-synchronous rounds -- Algorithm 4's
// swap of input and output queues, made device-wide -- and a pixel offers the
// feature it held at the end of the previous round, so round r is the dense
// operator
//     f_r(q) = argmin over p in N_G[q] of (d2(q, f_{r-1}(p)), f_{r-1}(p))
// (lexicographic: squared distance, then feature index) and the result does
// not depend on thread order.
//
// How: K rounds per tile visit (temporal blocking).  The image is cut into
// tiles of TE x TE pixels, TE = 64 - 2K.  A workgroup visits a tile: it loads
// the tile with a K-pixel halo (a 64 x 64 region) from the state after round r
// into LDS and runs K rounds there.  Round i leaves the pixels at least i away
// from the region's edge as the operator would, so after K rounds the tile is
// exactly at round r + K and goes to the other state buffer.  One step of the
// persistent kernel visits the listed tiles and ends in one grid barrier, so
// K rounds cost one barrier.  Which tiles a step must visit follows from two
// facts: a pixel's value only improves (its own previous feature is always a
// candidate), and a change travels at most one pixel per round.  So a tile can
// change during a step only if some pixel within K pixels of it changed in
// the last round of the previous step; such a change lists the tile that
// holds it and the neighbours within reach.  A tile that changed at all during
// a step is listed again, so that it rewrites its (then settled) values into
// the other buffer: a tile that is not visited holds equal values in both
// buffers, and every pixel a visit reads is at round r.
//
// A round in LDS is a push.  Only a pixel that changed in the previous round
// can improve a neighbour (the others' offers were weighed before), so the
// pixels of the previous round's change masks are gathered into a list and
// offer their feature to each neighbour: the offered (squared distance,
// feature) is one 64-bit key, compared with the neighbour's key and, where
// smaller, taken with an LDS 64-bit minimum.  Every lane holds its sources'
// features in registers before the first offer of a round, so a pixel offers
// what it held at the end of the previous round whatever the order; the
// minimum does not depend on the order either.
//
// Bound: 9 bytes a pixel have to move (30 us for 4096^2 at the copy rate); the
// time goes to a visit's serial chain -- in cycles 5 k to load, per round 1.4 k
// to list the sources and 0.8 k to push them, 5 k to store and list tiles --
// which four workgroups per CU (40 KB of keys each) hide in part, and to the
// slowest visit of each step.  Measured (30% features, whole calls one after
// another): 4096^2 1138 us, 389 x 517 246 us.  Before, a pull over the
// neighbourhood of every change (26 x 26 tiles, four rounds a visit, one wave each;
// eleven evaluations of nine candidates per changed pixel): 1515 and 516 us.
//
// The tiles of a step are a work list split into eight sub-lists, one per
// group of workgroups (one per XCD), appended to with one atomic per flush; a
// per-tile flag keeps a tile on a step's list once.  With more tiles than
// workgroups, a group visits its own sub-list (the neighbours of what it visited
// last, in its own L2) and its workgroups take items as they get to them:
// 4096^2 1190 us a call with items dealt round-robin over all workgroups, 1160
// with one counter for all, 1117 by group.
//
// State in memory is the feature's packed coordinates (y << 16 | x), 4 bytes
// per pixel.
#include "iwpp_device.hpp"
#include "iwpp_internal.hpp"

namespace iwpp {
namespace edt {

constexpr int K = kEdtHalo;        // rounds per step = halo width
constexpr int TE = kEdtTile;       // tile side
constexpr int R = TE + 2 * K;      // region side: one 64-bit mask word per row
constexpr int P = R + 2;           // LDS pitch: the region has a ring of pixels that never change around it
constexpr int kStageCap = 64;      // LDS work-list stage (iwpp_options.stage_depth caps it)
constexpr int kPart = 256;         // sources a wave lists at a time
constexpr uint32_t kTaken = 32;      // word of a count's cell with the items taken from the step's list
constexpr uint32_t kNoTile = 0xFFFFFFFFu;
constexpr uint32_t kMaxSteps = (1u << 20) / K;
static_assert(R == 64, "one mask bit per region column, one lane per region row");
static_assert(K % 4 == 0 && TE % 4 == 0, "16-byte chunks must not straddle the image's left edge or a tile's");
static_assert(K <= TE, "a change must reach no farther than the neighbouring tiles");
static_assert(K <= 8, "a change record's shortest word holds the columns a neighbour looks at");
static_assert(TE == kEdtTile && TE <= 64, "change records are one word of at most 64 bits per tile row");

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef short s2 __attribute__((ext_vector_type(2)));
typedef unsigned short u2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_yx(int y, int x) { return ((uint32_t)y << 16) | (uint32_t)x; }
__device__ __forceinline__ uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }

// Coordinate arithmetic of the state words, in two forms.
//
// Narrow (sides up to 32767): coordinates are signed 16-bit fields and "none"
// is (-32768, -32768).  A squared distance is one saturating packed 16-bit
// subtraction and one 2-term dot product; none's saturated distance,
// 2 * 32767^2, exceeds that of any real feature (coordinates are below 32767),
// and its packed value any real feature's, so it needs no special case.
//
// Wide (sides up to 46340, with (h-1)^2 + (w-1)^2 < 2^31 so that squared
// distances fit the int32 output): coordinates are unsigned 16-bit fields and
// none is all ones.  |dy|, |dx| come from packed maxima and minima, their
// squares sum in an unsigned dot product (below 2^32 for such sides), and
// none is given distance 2^32 - 1 explicitly.
template <bool kWide>
struct Coord;

template <>
struct Coord<false> {
  static constexpr uint32_t none = 0x80008000u;
  // Squared distance between q (real) and f (real or none).
  __device__ static __forceinline__ uint32_t d2(uint32_t q, uint32_t f) {
    const s2 e = __builtin_elementwise_sub_sat(__builtin_bit_cast(s2, q), __builtin_bit_cast(s2, f));
    // The three-operand dot product with a zero addend (the compiler's choice,
    // the accumulating form, needs a register cleared first).
    uint32_t r;
    asm("v_dot2_i32_i16 %0, %1, %1, 0" : "=v"(r) : "v"(__builtin_bit_cast(uint32_t, e)));
    return r;
  }
  // What the distances from q's neighbours to the real feature f are computed from.
  __device__ static __forceinline__ uint32_t base(uint32_t q, uint32_t f) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(s2, q) - __builtin_bit_cast(s2, f));
  }
  __device__ static __forceinline__ uint32_t d2_at(uint32_t b, uint32_t, uint32_t step) {
    const s2 e = __builtin_bit_cast(s2, b) + __builtin_bit_cast(s2, step);
    uint32_t r;
    asm("v_dot2_i32_i16 %0, %1, %1, 0" : "=v"(r) : "v"(__builtin_bit_cast(uint32_t, e)));
    return r;
  }
};

template <>
struct Coord<true> {
  static constexpr uint32_t none = 0xFFFFFFFFu;
  __device__ static __forceinline__ uint32_t real_d2(uint32_t q, uint32_t f) {
    const u2 a = __builtin_bit_cast(u2, q), b = __builtin_bit_cast(u2, f);
    const u2 e = __builtin_elementwise_max(a, b) - __builtin_elementwise_min(a, b);
    return __builtin_amdgcn_udot2(e, e, 0u, false);
  }
  __device__ static __forceinline__ uint32_t d2(uint32_t q, uint32_t f) {
    return f == none ? 0xFFFFFFFFu : real_d2(q, f);
  }
  __device__ static __forceinline__ uint32_t base(uint32_t q, uint32_t) { return q; }
  __device__ static __forceinline__ uint32_t d2_at(uint32_t b, uint32_t f, uint32_t step) {
    return real_d2(__builtin_bit_cast(uint32_t, __builtin_bit_cast(u2, b) + __builtin_bit_cast(u2, step)), f);
  }
};

struct TileRef {
  EdtJob j;
  int ty, tx;
};

__device__ __forceinline__ TileRef tile_ref(const EdtArgs& a, uint32_t t) {
  TileRef r;
  r.j = uniform(a.njobs == 1u ? a.job0 : a.jobs[a.tile_job[t]]);
  const uint32_t lt = t - r.j.tile_base;
  r.ty = (int)(lt / (uint32_t)r.j.tiles_x);
  r.tx = (int)(lt - (uint32_t)r.ty * (uint32_t)r.j.tiles_x);
  return r;
}

// Buffer resource over the image rows [row0, row0 + rows) of a per-pixel u32
// array, plus `pad` bytes after them (the state buffers are padded so that a
// 16-byte load cut by the end of the last row stays inside).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const uint32_t* base, const EdtJob& j, int row0, int rows,
                                                            uint32_t pad = 0u) {
  return make_rsrc(base + j.pix_base + (unsigned long long)row0 * (uint32_t)j.w, (uint32_t)rows * (uint32_t)j.w * 4u + pad);
}

// Offset that makes a raw buffer access fall outside every buffer (reads 0).
constexpr uint32_t kOutside = 0xFFFFFFF0u;
constexpr uint32_t kStatePad = 16u;  // readable bytes after the last pixel of a state buffer
static_assert(kStatePad <= kEdtStatePad, "state buffers must be padded");

// LDS of a workgroup.  key: (squared distance << 32 | feature) of every region
// pixel and the ring around it; pixels outside the image and the ring hold 0,
// which no offer is below, so they never change and need no bounds checks.
// chg: the pixels that changed in a round (bit = region column), for two
// consecutive rounds.  list: a wave's sources (region row << 6 | column).
// any[i & 1]: round i has a source.
template <int WPB>
struct WgLds {
  unsigned long long key[P * P];
  unsigned long long chg[2][R];
  uint16_t list[WPB][kPart];
  uint32_t any[2];
};

__device__ __forceinline__ int at(int row, int col) { return (row + 1) * P + col + 1; }

// Load the region of tile tr (rows and columns from K before the tile) from
// `src` into the keys: 16-byte chunks, all loads issued before the first is
// used; a chunk cut by the image's right edge is loaded whole (the state
// buffers are padded).
template <bool kWide, int WPB>
__device__ __forceinline__ void load_region(const uint32_t* src, const TileRef& tr, WgLds<WPB>& L) {
  const EdtJob& j = tr.j;
  const int ry0 = tr.ty * TE - K, rx0 = tr.tx * TE - K;
  const int row0 = ry0 > 0 ? ry0 : 0;
  const int row1 = ry0 + R < j.h ? ry0 + R : j.h;
  const __amdgpu_buffer_rsrc_t rs = rows_rsrc(src, j, row0, row1 - row0, kStatePad);
  constexpr int kPer = R * R / 4 / (kWave * WPB);
  const int t = local_copy((int)threadIdx.x), c = 4 * (t & 15), xs = rx0 + c;
  v4u v[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int y = ry0 + (t >> 4) + k * (4 * WPB);
    const bool ok = y >= 0 && y < j.h && xs >= 0 && xs < j.w;
    const uint32_t off = ok ? ((uint32_t)(y - row0) * (uint32_t)j.w + (uint32_t)xs) * 4u : kOutside;
    v[k] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, kSc1));
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int row = (t >> 4) + k * (4 * WPB), y = ry0 + row;
    const bool row_ok = y >= 0 && y < j.h;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int x = xs + b;
      const uint32_t f = v[k][b], d = Coord<kWide>::d2(pack_yx(y, x), f);
      const bool ok = row_ok && x >= 0 && x < j.w;
      L.key[at(row, c + b)] = ok ? ((unsigned long long)d << 32 | f) : 0ull;
    }
  }
}

// Which neighbouring tiles lie within K pixels of the marked pixels of a tile
// row (`m`, bit = tile column) -- 1 top, 2 bottom, 3 left, 4 right, 5
// top-left, 6 top-right, 7 bottom-left, 8 bottom-right -- and bit 0, the tile
// itself, if any is marked.
__device__ __forceinline__ uint32_t zone_bits(unsigned long long m, int row) {
  const bool any = m != 0ull, t = any && row < K, b = any && row >= TE - K;
  const bool l = (m & ((1ull << K) - 1ull)) != 0ull, r = (m >> (TE - K)) != 0ull;
  return (any ? 1u : 0u) | (t ? 2u : 0u) | (b ? 4u : 0u) | (l ? 8u : 0u) | (r ? 16u : 0u) | (t && l ? 32u : 0u) |
         (t && r ? 64u : 0u) | (b && l ? 128u : 0u) | (b && r ? 256u : 0u);
}

// The lanes' zone bits OR-ed over the wave.
__device__ __forceinline__ uint32_t any_zone(uint32_t zone) {
  uint32_t z = 0;
#pragma unroll
  for (int b = 0; b < 9; ++b)
    if (ballot((zone >> b) & 1u)) z |= 1u << b;
  return z;
}

constexpr unsigned long long kTileCols = ((1ull << TE) - 1ull) << K;  // region columns of the tile

// The offers of one source (region row << 6 | column, feature f) to its
// neighbours: taken where smaller than the neighbour's key, which marks the
// neighbour as changed in this round.
template <int CONN, bool kWide, int WPB>
__device__ __forceinline__ void push(WgLds<WPB>& L, unsigned long long* now, uint32_t e, uint32_t f, uint32_t q0) {
  constexpr int NC = CONN == 8 ? 8 : 4;
  constexpr int kDy[8] = {-1, 1, 0, 0, -1, -1, 1, 1}, kDx[8] = {0, 0, -1, 1, -1, 1, -1, 1};
  const int row = (int)(e >> 6), col = (int)(e & 63u);
  unsigned long long* k = &L.key[at(row, col)];
  const uint32_t q = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u2, q0) + __builtin_bit_cast(u2, pack_yx(row, col)));
  const uint32_t b = Coord<kWide>::base(q, f);
  // Four offers are on their way before the first answer is looked at; left to
  // itself the compiler waits four times for eight (7001 x 5003 with
  // 4-connectivity 2936 us, 2870; eight at once cost as many registers as they
  // save waits).
  uint32_t took[3] = {0u, 0u, 0u};  // by row: bit 0 left, 1 same column, 2 right
#pragma unroll
  for (int g = 0; g < NC; g += 4) {
    unsigned long long old[4];
    uint32_t d2[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int n = g + m;
      const uint32_t step = ((uint32_t)kDy[n] << 16) | ((uint32_t)kDx[n] & 0xffffu);
      d2[m] = Coord<kWide>::d2_at(b, f, step);
      old[m] = __hip_atomic_fetch_min(&k[kDy[n] * P + kDx[n]], (unsigned long long)d2[m] << 32 | f, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < 4; ++m)
      took[kDy[g + m] + 1] |= (old[m] > ((unsigned long long)d2[m] << 32 | f) ? 1u : 0u) << (kDx[g + m] + 1);
  }
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (took[d])  // never beyond the region: the ring takes nothing
      __hip_atomic_fetch_or(&now[row + d - 1], col > 0 ? (unsigned long long)took[d] << (col - 1) : (unsigned long long)took[d] >> 1,
                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// K rounds on the region in LDS.  Round i's sources are the pixels that
// changed in round i-1 (for round 1, chg[0]: the last round of the previous
// step, or the contour features of the image) at least i-1 away from the
// region's edge; a round without any ends the visit's work.  Each wave takes
// every WPB-th row, a lane every WPB-th pixel of a row, so that a long run of
// changes is walked by several lanes.  Per lane: the tile's pixels that
// changed (over the rounds) and the last round that changed one.
template <int CONN, bool kWide, int WPB>
__device__ __forceinline__ void relax_steps(WgLds<WPB>& L, const TileRef& tr, uint32_t& changed, uint32_t& last) {
  constexpr int kParts = (64 / WPB) * 64 / kPart, kPer = kPart / kWave;
  const int l = local_copy(lane()), w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int row = (l / WPB) * WPB + w;
  const uint32_t half = (WPB == 4 ? 0x11111111u : 0x01010101u) << (l % WPB);
  const unsigned long long mine = (unsigned long long)half << 32 | half;  // this lane's columns
  const unsigned long long own = row >= K && row < K + TE ? kTileCols : 0ull;
  const uint32_t q0 = pack_yx(tr.ty * TE - K, 0) | ((uint32_t)(tr.tx * TE - K) & 0xffffu);
  uint16_t* list = L.list[w];
#pragma unroll 1
  for (int i = 1; i <= K; ++i) {
    unsigned long long* now = L.chg[i & 1];
    const unsigned long long all = L.chg[(i - 1) & 1][row] & mine;
    if (l % WPB == 0) now[row] = 0ull;
    if (i > 1) {
      const uint32_t c = (uint32_t)__popcll(all & own);
      changed += c;
      if (c) last = (uint32_t)(i - 1);
    }
    const unsigned long long m = row >= i - 1 && row <= R - i ? all & (~0ull << (i - 1)) & (~0ull >> (i - 1)) : 0ull;
    uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
    const uint32_t c = (uint32_t)(__popc(lo) + __popc(hi)), incl = wave_incl_sum(c), n = readlane(incl, kWave - 1);
    if (n != 0u && l == 0) L.any[i & 1] = 1u;
    if (threadIdx.x == 0) L.any[(i + 1) & 1] = 0u;  // last read in round i-1, next set in round i+1
    uint32_t a = incl - c, b = a + (uint32_t)__popc(lo);
    const uint32_t r = (uint32_t)row << 6;
    uint32_t ent[kParts * kPer / 2], f[kParts * kPer];
    static_assert(kPer % 2 == 0, "two entries a register");  // (4096^2: one spills 7 more, 1085 us against 1061)
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
      if (p > 0 && __builtin_expect(n <= (uint32_t)(p * kPart), 1)) break;  // wave-uniform
      uint32_t x = lo, y = hi, ax = a - (uint32_t)(p * kPart), bx = b - (uint32_t)(p * kPart);
      while (x | y) {  // both halves of the row at once
        if (x) {
          if (ax < (uint32_t)kPart) list[ax] = (uint16_t)(r | (uint32_t)__builtin_ctz(x));
          x &= x - 1u;
          ++ax;
        }
        if (y) {
          if (bx < (uint32_t)kPart) list[bx] = (uint16_t)(r | 32u | (uint32_t)__builtin_ctz(y));
          y &= y - 1u;
          ++bx;
        }
      }
      wave_sync();
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        if (q > 0 && n <= (uint32_t)(p * kPart + q * kWave)) break;
        const uint32_t idx = (uint32_t)(q * kWave + l);
        const uint32_t e = (uint32_t)(p * kPart) + idx < n ? (uint32_t)list[idx] : 0u;
        ent[(p * kPer + q) / 2] = q & 1 ? ent[(p * kPer + q) / 2] | e << 16 : e;
        f[p * kPer + q] = (uint32_t)L.key[at((int)(e >> 6), (int)(e & 63u))];
      }
      wave_sync();
    }
    __syncthreads();  // every source is read, the round's masks are clear
    const uint32_t any = L.any[i & 1];
#pragma unroll
    for (int q = 0; q < kParts * kPer; ++q) {
      if (n <= (uint32_t)(q * kWave)) break;
      if ((uint32_t)(q * kWave + l) < n) push<CONN, kWide, WPB>(L, now, ent[q / 2] >> (16 * (q & 1)) & 0xffffu, f[q], q0);
    }
    __syncthreads();
    if (any == 0u) break;  // (asked for here, the answer is not waited for)
  }
  const uint32_t c = (uint32_t)__popcll(L.chg[K & 1][row] & mine & own);
  changed += c;
  if (c) last = (uint32_t)K;
}

// Region change mask (one 64-bit word per region row, bit = region column)
// of the pixels that changed in the last round of step m-1.  Every such pixel
// lies in a tile visited in step m-1, which recorded its last-round changes
// (`record_changes`) under that step's parity with stamp m-1; a tile whose
// stamp differs did not change.  One wave, lane = region row: the stamps and
// row words of three tiles (left neighbour, own column, right neighbour).
// Split in two so that the loads are in flight with the region's.
//
// Row y's word of a tile column is word y of the column's run (`edt_mark_words`).
// Words of every width are read alike, as the 8 bytes that begin there, and cut to
// the column's bits, with no branch on the width or on the image's edges (7001 x
// 5003 with 4-connectivity 2750 us; loads of each width behind branches 2912; 48
// words of 8 bytes a tile, whatever its size, 2723; 4096^2 1119, 1118 and 1125).
__device__ __forceinline__ int mark_cols(const EdtJob& j, int tx) { return tx + 1 < j.tiles_x ? TE : j.w - tx * TE; }
__device__ __forceinline__ uint32_t mark_offset(const EdtJob& j, int tx, int y) {
  return (uint32_t)tx * (uint32_t)j.h * 8u + ((uint32_t)y << edt_mark_shift(mark_cols(j, tx)));
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t marks_rsrc(const EdtArgs& a, const EdtJob& j, uint32_t par) {
  // No image has more than tiles_x full columns' runs; 8 bytes are read at the last word.
  return make_rsrc(a.marks + (size_t)par * a.mark_words + j.mark_base, (uint32_t)j.tiles_x * (uint32_t)j.h * 8u + 8u);
}

// Every lane with `ok`: m as row y's word, by the one of four stores of its width;
// the others go outside the buffer.
__device__ __forceinline__ void store_mark(const EdtArgs& a, const TileRef& tr, uint32_t par, bool ok, int y,
                                           unsigned long long m) {
  const __amdgpu_buffer_rsrc_t rm = marks_rsrc(a, tr.j, par);
  const int sh = edt_mark_shift(mark_cols(tr.j, tr.tx));
  const uint32_t off = ok ? mark_offset(tr.j, tr.tx, y) : kOutside;
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, m), rm, sh == 3 ? off : kOutside, 0, kSc1);
  __builtin_amdgcn_raw_buffer_store_b32((uint32_t)m, rm, sh == 2 ? off : kOutside, 0, kSc1);
  __builtin_amdgcn_raw_buffer_store_b16((uint16_t)m, rm, sh == 1 ? off : kOutside, 0, kSc1);
  __builtin_amdgcn_raw_buffer_store_b8((uint8_t)m, rm, sh == 0 ? off : kOutside, 0, kSc1);
}

struct PrevChanges {
  uint32_t stamp[3];
  unsigned long long word[3];
};

__device__ __forceinline__ void prev_step_issue(const EdtArgs& a, const TileRef& tr, uint32_t m, PrevChanges& pc) {
  const EdtJob& j = tr.j;
  const uint32_t par = (m - 1u) & 1u;
  const int y = tr.ty * TE - K + lane();
  const bool row_ok = y >= 0 && y < j.h;
  const int ty = row_ok ? y / TE : 0;
  const __amdgpu_buffer_rsrc_t rm = marks_rsrc(a, j, par);
  const __amdgpu_buffer_rsrc_t rt =
      make_rsrc(a.stamps + (size_t)par * a.ntiles + j.tile_base, (uint32_t)j.tiles_y * (uint32_t)j.tiles_x * 4u);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int tx = tr.tx + d - 1;
    const bool ok = row_ok && tx >= 0 && tx < j.tiles_x;
    const uint32_t so = ok ? (uint32_t)(ty * j.tiles_x + tx) * 4u : kOutside, off = ok ? mark_offset(j, tx, y) : kOutside;
    pc.stamp[d] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rt, so, 0, kSc1);
    pc.word[d] = __builtin_bit_cast(unsigned long long, __builtin_amdgcn_raw_buffer_load_b64(rm, off, 0, kSc1));
  }
}

__device__ __forceinline__ void prev_step_finish(const TileRef& tr, uint32_t m, const PrevChanges& pc,
                                                 unsigned long long* M) {
  unsigned long long v = 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (pc.stamp[d] != m - 1u) continue;
    // (the left column is a full one, and of the right one K columns are wanted, no more than its shortest word has)
    const unsigned long long w = d == 1 ? pc.word[d] & ((1ull << mark_cols(tr.j, tr.tx)) - 1ull) : pc.word[d];
    // region column rx <-> tile column rx - K - (d - 1) * TE
    v |= d == 0 ? (w >> (TE - K)) : (d == 1 ? (w << K) : ((w & ((1ull << K) - 1ull)) << (K + TE)));
  }
  M[lane()] = v;
}

// Record this visit's last-round changes of the tile (rows and columns
// [K, K + TE) of the round-K mask word `m` of region row lane()) and stamp
// them with step `step`.
__device__ __forceinline__ void record_changes(const EdtArgs& a, const TileRef& tr, uint32_t t, uint32_t step,
                                               unsigned long long m) {
  const int l = lane(), y = tr.ty * TE + l - K;
  const uint32_t par = step & 1u;
  store_mark(a, tr, par, l >= K && l < K + TE && y < tr.j.h, y, (m & kTileCols) >> K);
  if (l == 0) cstore(a.stamps + (size_t)par * a.ntiles + t, step);
}

// Store the tile (region rows and columns [K, K + TE)) to `dst`.
template <int WPB>
__device__ __forceinline__ void store_tile(const WgLds<WPB>& L, uint32_t* dst, const TileRef& tr) {
  const EdtJob& j = tr.j;
  const int y0 = tr.ty * TE, x0 = tr.tx * TE;
  const int row1 = y0 + TE < j.h ? y0 + TE : j.h;
  const __amdgpu_buffer_rsrc_t rs = rows_rsrc(dst, j, y0, row1 - y0);
  constexpr int kCpr = TE / 4;
  for (int idx = local_copy((int)threadIdx.x); idx < TE * kCpr; idx += kWave * WPB) {
    const int cy = idx / kCpr, cx = 4 * (idx - cy * kCpr);
    const int y = y0 + cy, x = x0 + cx;
    if (y >= j.h || x >= j.w) continue;
    const unsigned long long* k = &L.key[at(cy + K, cx + K)];
    const v4u v = {(uint32_t)k[0], (uint32_t)k[1], (uint32_t)k[2], (uint32_t)k[3]};
    const uint32_t off = ((uint32_t)cy * (uint32_t)j.w + (uint32_t)x) * 4u;
    if (x + 4 <= j.w) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v), rs, off, 0, kSc1);
    } else {
#pragma unroll
      for (int b = 0; b < 3; ++b)
        if (x + b < j.w) __builtin_amdgcn_raw_buffer_store_b32(v[b], rs, off + 4u * b, 0, kSc1);
    }
  }
}

// The list of step m+1 while step m runs (m = 0 for the initial list): the
// parity's flags and the sub-list of this workgroup's group.
struct Next {
  uint32_t* flags;
  uint32_t* list;
  uint32_t* count;
};

__device__ __forceinline__ Next next_frontier(const EdtArgs& a, uint32_t m) {
  const uint32_t par = (m + 1u) & 1u, shard = blockIdx.x & (uint32_t)(kShards - 1);
  Next n;
  n.flags = a.flags + (size_t)par * a.ntiles;
  n.list = a.lists + ((size_t)par * kShards + shard) * a.ntiles;
  n.count = shard_count(a.counts, (m + 1u) % 3u, shard);
  return n;
}

// List, for the next step, the tiles named by zone mask z of tile tr: itself
// (bit 0) and the neighbours of bits 1..8.  Lanes 0..8 of the wave each
// handle one candidate.
__device__ __forceinline__ void mark_reach(const EdtArgs& a, WaveStage& s, const Next& nx, const TileRef& tr, uint32_t z,
                                           uint32_t* appended) {
  const int l = local_copy(lane());
  int dy = 0, dx = 0;
  bool want = false;
  if (l == 0) {
    want = (z & 1u) != 0u;
  } else if (l <= 8) {
    // lanes 1..8: top, bottom, left, right, top-left, top-right, bottom-left, bottom-right
    const int k = l - 1;
    want = (z & (k < 4 ? (2u << k) : (32u << (k - 4)))) != 0u;
    dy = k == 0 ? -1 : (k == 1 ? 1 : (k < 4 ? 0 : (k < 6 ? -1 : 1)));
    dx = k < 2 ? 0 : (k == 2 ? -1 : (k == 3 ? 1 : ((k & 1) ? 1 : -1)));
  }
  const int ny = tr.ty + dy, nx_ = tr.tx + dx;
  want = want && ny >= 0 && ny < tr.j.tiles_y && nx_ >= 0 && nx_ < tr.j.tiles_x;
  shard_mark(s, want, tr.j.tile_base + (uint32_t)(ny * tr.j.tiles_x + nx_), nx.flags, nx.list, nx.count, a.ntiles, a.ovf,
             appended);
}

// Initial state (features carry themselves, everything else none), the
// contour-feature count (Algorithm 6's initial queue), and what the first
// step's list is made of: round 1 changes exactly the non-features next to a
// feature, so their tiles and the neighbours within K pixels are visited; a
// tile's word in the odd stamps says which (`kZoneWord` | zone bits; no step
// number has that bit, so no later step takes it for a stamp).  The contour
// features are every tile's step-0 change record, from which the first step's
// round 1 takes its sources.  Clears the flags of both parities.
//
// A workgroup per tile, lane = column (lane 0 the column before the tile) for
// the pixels and lane = row for the masks: a row's ballot goes through LDS to
// the lane of that row in every wave, which tests all rows at once.  (One
// scalar mask computation per row instead kept the scalar unit busy for 1050
// instructions a wave, and each tile's atomics on flags and list its workgroups'
// ends: 75 us of a 4096 x 4096 transform.  Now 50, and 5 for `k_list`.)
//
// Both buffers need the initial state where the first step does not visit; a
// tile with a round-1 change lists itself, and its visit writes the second.
constexpr uint32_t kZoneWord = 0x80000000u;

template <int CONN, bool kWide>
__global__ __launch_bounds__(256) void k_init(EdtArgs a) {
  constexpr int kRows = TE + 2, kPer = (kRows + 3) / 4;  // rows with the one above and the one below; per wave
  __shared__ unsigned long long feat_sh[kRows];
  static_assert(kRows <= 64, "a lane per row and per column, with one to each side");
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), l = lane();
  const uint32_t t = blockIdx.x;
  const TileRef tr = tile_ref(a, t);
  const EdtJob& j = tr.j;
  const int y0 = tr.ty * TE - 1, x = tr.tx * TE - 1 + l;
  const bool in_x = x >= 0 && x < j.w && l < kRows;
  uint8_t px[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = 4 * k + w, y = y0 + r;
    px[k] = in_x && r < kRows && y >= 0 && y < j.h ? j.bin[(size_t)y * (uint32_t)j.w + (uint32_t)x] : (uint8_t)1;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = 4 * k + w;
    const unsigned long long f = ballot(px[k] == 0);
    if (r < kRows && l == 0) feat_sh[r] = f;
  }
  __syncthreads();
  // Lane = row l of feat_sh; what lies outside the image is neither feature nor pixel.
  const unsigned long long cols = ballot(in_x), own = ((1ull << TE) - 1ull) << 1;
  auto rows = [&](int r, unsigned long long& f, unsigned long long& o) {
    const bool ok = r >= 0 && r < kRows && y0 + r >= 0 && y0 + r < j.h;
    f = ok ? feat_sh[r] : 0ull;
    o = ok ? cols & ~f : 0ull;
  };
  unsigned long long f0, f1, f2, o0, o1, o2;
  rows(l - 1, f0, o0);
  rows(l, f1, o1);
  rows(l + 1, f2, o2);
  auto near = [&](unsigned long long u, unsigned long long m, unsigned long long d) {  // pixels with a marked neighbour
    if (CONN == 4) return u | d | (m << 1) | (m >> 1);
    const unsigned long long v = u | m | d;
    return (v << 1) | (v >> 1) | u | d;
  };
  // Round 0's changes as round 1 sees them: only the contour features offer
  // anything new (a feature keeps itself; a pixel away from every feature
  // stays none).
  const bool mine = l >= 1 && l <= TE;
  const unsigned long long ct = mine ? f1 & near(o0, o1, o2) & own : 0ull;
  const unsigned long long first = mine ? o1 & near(f0, f1, f2) & own : 0ull;
  const uint32_t zone = any_zone(zone_bits(first >> 1, l - 1));
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = 4 * k + w, y = y0 + r;
    if (r >= 1 && r <= TE && y < j.h && ((cols & own) >> l & 1ull)) {
      const uint32_t v = px[k] == 0 ? pack_yx(y, x) : Coord<kWide>::none;
      const size_t p = j.pix_base + (size_t)y * (uint32_t)j.w + (uint32_t)x;
      a.feat0[p] = v;
      if (!(zone & 1u)) a.feat1[p] = v;
    }
  }
  if (w == 0) {
    store_mark(a, tr, 0u, mine && y0 + l < j.h, y0 + l, ct >> 1);
    const uint32_t contour = wave_incl_sum((uint32_t)__popcll(ct));
    if (l == kWave - 1 && contour) {
      stat_add(a.stats, kStatSeeds, contour);
      stat_add(a.stats, kStatItems, contour);  // the first frontier
    }
    if (l == 0) {
      cstore(a.stamps + t, 0u);
      cstore(a.stamps + a.ntiles + t, kZoneWord | zone);
      cstore(a.flags + t, 0u);
    }
  }
}

// The first step's list from the tiles' zone words: a tile is listed if round
// 1 changes one of its pixels or one within K pixels of it.
__global__ void k_list(EdtArgs a) {
  const int w = (int)(threadIdx.x / kWave);
  const Next nx = next_frontier(a, 0u);  // step 1's list
  const uint32_t* zones = a.stamps + a.ntiles;
  for (uint32_t t0 = (blockIdx.x * 4u + (uint32_t)w) * (uint32_t)kWave; t0 < a.ntiles; t0 += gridDim.x * 256u) {
    const uint32_t t = t0 + (uint32_t)lane();
    bool want = false;
    if (t < a.ntiles) {
      const EdtJob& j = a.njobs == 1u ? a.job0 : a.jobs[a.tile_job[t]];
      const int ty = (int)((t - j.tile_base) / (uint32_t)j.tiles_x), tx = (int)((t - j.tile_base) % (uint32_t)j.tiles_x);
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy) {
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx) {
          if (ty + dy < 0 || ty + dy >= j.tiles_y || tx + dx < 0 || tx + dx >= j.tiles_x) continue;
          // The bit with which that tile names this one: the zone opposite to where it lies.
          const uint32_t bit = dy == 0 ? (dx == 0 ? 1u : (dx < 0 ? 16u : 8u))
                                       : (dx == 0 ? (dy < 0 ? 4u : 2u) : (dy < 0 ? (dx < 0 ? 256u : 128u) : (dx < 0 ? 64u : 32u)));
          want = want || (zones[(int)t + dy * j.tiles_x + dx] & bit) != 0u;
        }
      }
      nx.flags[t] = want ? 1u : 0u;
    }
    const unsigned long long m = ballot(want);
    if (m == 0ull) continue;
    uint32_t at0 = 0;
    if (lane() == 0) at0 = atomic_add(nx.count, (uint32_t)__popcll(m));
    at0 = readlane(at0, 0);
    if (want) cstore(nx.list + at0 + mbcnt(m), t);  // each tile once: a sub-list holds them all
  }
}

// An item beyond the dealt ones of another group's sub-list (cnt[x] items each,
// `stride` apart), from the first group after `grp` that has one; one wave.
// Ends: each pass without an item has seen a counter grow past its sub-list.
__device__ __forceinline__ uint32_t steal(const uint32_t* lists, uint32_t stride, uint32_t* taken, const uint32_t* cnt,
                                          uint32_t grp) {
  const uint32_t x = (grp + 1u + (uint32_t)lane()) % kXcds, dealt = xcd_groups(x);
  const bool other = lane() < (int)kXcds - 1 && cnt[x] > dealt;
  if (ballot(other) == 0ull) return kNoTile;
  for (;;) {
    const unsigned long long left = ballot(other && dealt + cload(taken + 64u * x) < cnt[x]);
    if (left == 0ull) return kNoTile;
    const int src = __builtin_ctzll(left);
    uint32_t t = kNoTile;
    if (lane() == src) {
      const uint32_t i = dealt + atomic_add(taken + 64u * x, 1u);
      if (i < cnt[x]) t = cload(lists + (size_t)x * stride + i);
    }
    t = readlane(t, src);
    if (t != kNoTile) return t;
  }
}

// A workgroup of WPB waves per tile visit; four workgroups of four waves fit a
// CU's LDS, two of eight its registers.
template <int CONN, bool kWide, int WPB>
__global__ __launch_bounds__(64 * WPB, 4) void k_rounds(EdtArgs a) {
  __shared__ WgLds<WPB> L;
  __shared__ uint32_t stage_mem[kStageCap];
  __shared__ uint32_t cnt[kShards];
  __shared__ uint32_t last_sh;  // the visit's last round with a change
  __shared__ uint32_t next_sh;  // the tile to visit next
  __shared__ uint32_t appended_sh;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t depth = a.stage_depth > 0u && a.stage_depth < (uint32_t)kStageCap ? a.stage_depth : (uint32_t)kStageCap;
  WaveStage s = {stage_mem, depth, 0u};  // wave 0's
  for (int i = (int)threadIdx.x; i < P * P; i += kWave * WPB) L.key[i] = 0ull;  // the ring stays so
  if (threadIdx.x == 0) last_sh = appended_sh = L.any[0] = L.any[1] = 0u;
  Appended app = {&appended_sh, cnt, nullptr, 0u};
  shard_counts(a.counts, 1u, a.ntiles, cnt);  // `k_list`'s
  __syncthreads();
  uint32_t gen = 0, nclk = 0;
  unsigned long long changed = 0, visits = 0;
  uint32_t last_round = 0;  // this workgroup's last round with a change (wave 0)
  clock_stamp(a.clock, nclk);
  for (uint32_t m = 1;; ++m) {
    uint32_t n = 0;
    for (int x = 0; x < kShards; ++x) n += cnt[x];
    if (n == 0u) break;
    round_work(a.clock, m - 1u, n);
    if (m >= kMaxSteps) {  // safety limit: report instead of spinning on a logic error
      if (blockIdx.x == 0 && threadIdx.x == 0) stat_add(a.stats, kStatError, 1ull);
      break;
    }
    // The counts of step m+2 are reused: clear them now (they were last read
    // at the start of step m-1 and are next appended to in step m+1, after
    // this step's barrier).
    if (blockIdx.x == 0 && threadIdx.x < (unsigned)kShards) {
      cstore(shard_count(a.counts, (m + 2u) % 3u, threadIdx.x), 0u);
      cstore(shard_count(a.counts, (m + 2u) % 3u, threadIdx.x) + kTaken, 0u);
    }
    const uint32_t* rd = (m & 1u) ? a.feat0 : a.feat1;  // buffer (m-1)&1
    uint32_t* wr = (m & 1u) ? a.feat1 : a.feat0;        // buffer m&1
    const uint32_t par = m & 1u;
    const uint32_t* lists = a.lists + (size_t)par * kShards * a.ntiles;
    uint32_t* flg = a.flags + (size_t)par * a.ntiles;
    const Next nx = next_frontier(a, m);
    // At most one item per workgroup: item b goes to workgroup b, which spreads
    // them over the CUs.  Otherwise a group (XCD) takes its own sub-list, where
    // the neighbours of the tiles it visited last are: the first items by rank,
    // the others from the sub-list's counter as its workgroups get to them, and
    // at its end those of the other groups.  The next item is taken while the
    // current tile is visited.
    const bool sparse = n <= gridDim.x;
    const uint32_t grp = blockIdx.x % kXcds, rank = blockIdx.x / kXcds, dealt = xcd_groups(grp);
    uint32_t* taken = shard_count(a.counts, m % 3u, 0u) + kTaken;
    uint32_t t = kNoTile;
    if (sparse) {
      if (blockIdx.x < n) t = shard_item(lists, a.ntiles, cnt, blockIdx.x);
    } else if (rank < cnt[grp]) {
      t = cload(lists + (size_t)grp * a.ntiles + rank);
    } else {
      if (w == 0) {
        const uint32_t t0 = steal(lists, a.ntiles, taken, cnt, grp);
        if (lane() == 0) next_sh = t0;
      }
      __syncthreads();
      t = next_sh;
    }
    t = readlane(t, 0);
    while (t != kNoTile) {
      uint32_t i = cnt[grp];
      if (!sparse && threadIdx.x == 0 && i > dealt) i = dealt + atomic_add(taken + 64u * grp, 1u);
      const TileRef tr = tile_ref(a, t);
      PrevChanges pc;
      if (w == 0) {
        if (lane() == 0) cstore(flg + t, 0u);
        prev_step_issue(a, tr, m, pc);
      }
      load_region<kWide, WPB>(rd, tr, L);
      if (w == 0) prev_step_finish(tr, m, pc, L.chg[0]);
      uint32_t t_next = kNoTile;
      if (threadIdx.x == 0 && i < cnt[grp]) t_next = cload(lists + (size_t)grp * a.ntiles + i);
      __syncthreads();
      uint32_t c = 0, lr = 0;
      relax_steps<CONN, kWide, WPB>(L, tr, c, lr);
      changed += c;
      if (lr) atomicMax(&last_sh, lr);
      if (w == 0 && !sparse) {
        t_next = readlane(t_next, 0);
        if (t_next == kNoTile) t_next = steal(lists, a.ntiles, taken, cnt, grp);
        if (lane() == 0) next_sh = t_next;
      }
      store_tile<WPB>(L, wr, tr);
      __syncthreads();
      if (w == 0) {
        visits++;
        const unsigned long long mk = L.chg[K & 1][lane()];
        record_changes(a, tr, t, m, mk);
        const uint32_t lw = readlane(last_sh, 0);
        wave_sync();
        if (lane() == 0) last_sh = 0u;
        if (lw) last_round = umax32(last_round, (m - 1u) * (uint32_t)K + lw);
        const int row = lane() - K;
        uint32_t z = any_zone(row >= 0 && row < TE ? zone_bits((mk & kTileCols) >> K, row) : 0u);
        if (lw) z |= 1u;
        mark_reach(a, s, nx, tr, z, &appended_sh);
      }
      if (sparse) break;
      __syncthreads();  // LDS is reloaded by the next visit
      t = readlane(next_sh, 0);
    }
    if (w == 0) shard_flush(s, nx.list, nx.count, a.ntiles, nx.flags, a.ovf, &appended_sh);
    if (!grid_barrier(a.bar, gen, a.stats, &app)) return;  // leaves the next step's list lengths in cnt
    clock_stamp(a.clock, nclk);
  }
  // Both buffers now agree everywhere; write the outputs.  A wave takes 256
  // pixels of a row at a time, four per lane.
  const uint32_t nw = gridDim.x * WPB;
  for (uint32_t jj = 0; jj < a.njobs; ++jj) {
    const EdtJob j = uniform(a.njobs == 1u ? a.job0 : a.jobs[jj]);
    const uint32_t segs = ((uint32_t)j.w + 255u) / 256u, items = segs * (uint32_t)j.h;
    for (uint32_t i = blockIdx.x * WPB + (uint32_t)w; i < items; i += nw) {
      const uint32_t y = i / segs, x = (i - y * segs) * 256u + 4u * (uint32_t)lane();
      if (x >= (uint32_t)j.w) continue;
      const __amdgpu_buffer_rsrc_t rf = rows_rsrc(a.feat0, j, (int)y, 1, kStatePad);
      const __amdgpu_buffer_rsrc_t rd = make_rsrc(j.sqdist + (size_t)y * (uint32_t)j.w, (uint32_t)j.w * 4u);
      const __amdgpu_buffer_rsrc_t rn = make_rsrc(j.nearest + (size_t)y * (uint32_t)j.w, (uint32_t)j.w * 4u);
      const v4u f = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rf, 4u * x, 0, kSc1));
      v4i d, nr;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const bool none = f[b] == Coord<kWide>::none;
        d[b] = none ? -1 : (int)Coord<kWide>::d2(pack_yx((int)y, (int)x + b), f[b]);
        nr[b] = none ? -1 : (int)((f[b] >> 16) * (uint32_t)j.w + (f[b] & 0xffffu));
      }
      if (x + 4u <= (uint32_t)j.w) {
        __builtin_amdgcn_raw_buffer_store_b128(d, rd, 4u * x, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(nr, rn, 4u * x, 0, 0);
      } else {
#pragma unroll
        for (int b = 0; b < 3; ++b)
          if (x + (uint32_t)b < (uint32_t)j.w) {
            __builtin_amdgcn_raw_buffer_store_b32((uint32_t)d[b], rd, 4u * (x + (uint32_t)b), 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32((uint32_t)nr[b], rn, 4u * (x + (uint32_t)b), 0, 0);
          }
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) changed += __shfl_xor(changed, o);
  if (lane() == 0) {
    stat_add(a.stats, kStatItems, changed);  // pixels changed in a round join the next frontier
    stat_add(a.stats, kStatUpdates, changed);
    if (w == 0) {
      stat_add(a.stats, kStatSweeps, visits);
      // Rounds: the last round in which any pixel changed -- a maximum, kept in
      // shard 0 so that the host's sum over the shards leaves it unchanged.
      if (last_round) atomic_max(a.stats + kStatRounds, (unsigned long long)last_round);
    }
  }
}

// Image of every global tile, by binary search over the images' first tiles.
__global__ void k_tile_job(const EdtJob* jobs, uint32_t njobs, uint32_t* tile_job, uint32_t ntiles) {
  for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < ntiles; t += gridDim.x * blockDim.x) {
    uint32_t lo = 0, hi = njobs;
    while (hi - lo > 1u) {
      const uint32_t mid = (lo + hi) >> 1;
      if (jobs[mid].tile_base <= t) lo = mid; else hi = mid;
    }
    tile_job[t] = lo;
  }
}

}  // namespace edt

int edt_launch(const EdtArgs& a, int conn, int persistent_blocks, hipStream_t stream, Recorder* rec, const char** err) {
  using namespace edt;
  if (a.njobs > 1u) {
    const uint32_t b = (a.ntiles + 255u) / 256u;
    hipLaunchKernelGGL(k_tile_job, dim3(b < 1024u ? b : 1024u), dim3(256), 0, stream, a.jobs, a.njobs, a.tile_job, a.ntiles);
    if (hipGetLastError() != hipSuccess) {
      *err = "tile map launch failed";
      return -1;
    }
  }
  const uint32_t init_blocks = a.ntiles;
  rec->begin(4, stream);
  if (conn == 8 && !a.wide)
    hipLaunchKernelGGL((k_init<8, false>), dim3(init_blocks), dim3(256), 0, stream, a);
  else if (conn == 8)
    hipLaunchKernelGGL((k_init<8, true>), dim3(init_blocks), dim3(256), 0, stream, a);
  else if (!a.wide)
    hipLaunchKernelGGL((k_init<4, false>), dim3(init_blocks), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((k_init<4, true>), dim3(init_blocks), dim3(256), 0, stream, a);
  const uint32_t list_blocks = (a.ntiles + 255u) / 256u;
  hipLaunchKernelGGL(k_list, dim3(list_blocks < 1024u ? list_blocks : 1024u), dim3(256), 0, stream, a);
  rec->end(stream);
  if (hipGetLastError() != hipSuccess) {
    *err = "EDT init launch failed";
    return -1;
  }
  int dev = 0, per_cu = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    *err = "device query failed";
    return -1;
  }
  const int wpb = (int)edt_waves((int32_t)a.wg_waves, persistent_blocks, a.ntiles, cus);
  void* fn;
  if (wpb == 8)
    fn = conn == 8 ? (a.wide ? reinterpret_cast<void*>(&k_rounds<8, true, 8>) : reinterpret_cast<void*>(&k_rounds<8, false, 8>))
                   : (a.wide ? reinterpret_cast<void*>(&k_rounds<4, true, 8>) : reinterpret_cast<void*>(&k_rounds<4, false, 8>));
  else
    fn = conn == 8 ? (a.wide ? reinterpret_cast<void*>(&k_rounds<8, true, 4>) : reinterpret_cast<void*>(&k_rounds<8, false, 4>))
                   : (a.wide ? reinterpret_cast<void*>(&k_rounds<4, true, 4>) : reinterpret_cast<void*>(&k_rounds<4, false, 4>));
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64 * wpb, 0) != hipSuccess || per_cu < 1) {
    *err = "occupancy query failed";
    return -1;
  }
  uint32_t blocks = persistent_grid(fn, per_cu, cus, wpb == 4 ? 4 : 2);
  if (persistent_blocks > 0 && (uint32_t)persistent_blocks < blocks) blocks = (uint32_t)persistent_blocks;
  EdtArgs args = a;
  void* kargs[] = {&args};
  rec->begin(5, stream);
  const hipError_t le = launch_persistent(fn, blocks, kargs, stream, 64 * wpb);
  rec->end(stream);
  if (le != hipSuccess) {
    *err = "EDT rounds launch failed";
    return -1;
  }
  return 0;
}

uint32_t persistent_grid(const void* fn, int per_cu, int cus, int max_per_cu) {
  hipFuncAttributes fa{};
  int lim = per_cu < max_per_cu ? per_cu : max_per_cu;
  if (hipFuncGetAttributes(&fa, fn) == hipSuccess && fa.sharedSizeBytes > 0) {
    const int by_lds = (int)((160u * 1024u) / (unsigned)fa.sharedSizeBytes);  // LDS per CU
    if (by_lds < lim) lim = by_lds;
  }
  if (lim < 1) lim = 1;
  return (uint32_t)lim * (uint32_t)cus;
}

hipError_t launch_persistent(const void* fn, uint32_t blocks, void** args, hipStream_t s, uint32_t threads) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) == hipSuccess && cs == hipStreamCaptureStatusActive)
    return hipLaunchKernel(fn, dim3(blocks), dim3(threads), args, 0, s);
  return hipLaunchCooperativeKernel(fn, dim3(blocks), dim3(threads), args, 0, s);
}

// Zero two ranges of 32-bit words with one kernel (no memset node, so the sequence
// can be captured into a graph).
__global__ void k_zero(uint32_t* p, size_t n, uint32_t* q, size_t m) {
  const size_t i0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
  for (size_t i = i0; i < n; i += step) p[i] = 0u;
  for (size_t i = i0; i < m; i += step) q[i] = 0u;
}

int zero_words(uint32_t* p, size_t nwords, hipStream_t stream, uint32_t* q, size_t mwords) {
  size_t blocks = ((nwords > mwords ? nwords : mwords) + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  if (blocks == 0) return 0;
  hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, stream, p, nwords, q, mwords);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace iwpp
