// Grayscale morphological reconstruction by dilation on gfx950.
//
// What is computed (Sec. 2.1): rho_I(J), the limit of the elementary geodesic
// dilation J(p) <- max{J(q) : q in N_G(p) U {p}} ^ I(p).  The result is unique,
// so any schedule of valid updates that reaches stability gives identical
// bytes (the paper's exactness argument for Algorithm 5, which does hold here).
//
// How (the steps of Algorithm 5, re-planned for CDNA4).  One persistent,
// cooperative kernel runs in rounds (the queue swap of Algorithm 4); a round
// visits tiles, one wave per 64x64 tile held in LDS with a one-pixel halo:
//   round 0  -- the seed pass: every tile is loaded from the marker (clamped
//               to the mask) and swept with Algorithm 5's raster and
//               anti-raster scans, split into row-wise and column-wise
//               sweeps (lane = row or column), until it is locally stable
//               or a cap of sweep iterations is reached;
//   round r  -- each tile flagged in round r-1 is loaded from the current
//               image, swept the same way and written back.
// After a visit the wave flags each neighbouring tile that a border change
// can still raise (Algorithm 5's propagation condition, J(q) < J(p) and
// J(q) < I(q), tested against the halo as loaded), and the tile itself if the
// sweep cap stopped it.  This replaces Algorithm 5's dense seed detection: in
// round 0 a halo pixel holds the neighbour's initial value, and a border pixel
// that did not rise was seen with that same value by the neighbour's own
// sweep, so only risen border pixels can leave a seed across a tile edge.
//
// The tile frontier of a round is a work list split into eight sub-lists, one
// per group of workgroups (one per XCD): a wave stages its appends in LDS and
// flushes them with one atomic on its group's counter, a per-tile flag keeps a
// tile on a round's list once, and in the next round an XCD visits its own
// sub-list, cut into one share per workgroup whose waves take tiles as they get
// to them.  With a capacity (the paper's fixed-size global queue, Sec. 3.2) the list is one
// sub-list of that size: an append past it is dropped and flagged, and the
// next round becomes a full round that visits every tile holding a raisable
// pixel of the current image, which is a valid restart point because every
// intermediate image is (Sec. 3.2: re-running from a partial output gives the
// same answer).
//
// The value updates are max-then-min of bytes; the per-tile state is owned by
// exactly one wave at a time (a tile is on a round's list at most once), so no
// atomics touch pixels.  Halo reads may see a neighbour mid-update; any value
// they see is a valid lower bound, and a border change always re-lists the
// neighbour for the next round, which then reads it after a grid barrier.
//
// Bound: three bytes a pixel have to move (158 us for 16384^2 at the copy rate);
// the time goes to the scans' dependence chains, which four waves per SIMD (9
// KiB of LDS and 128 registers each) do not hide -- VALU issue is a little over
// half -- and, with few tiles, to one visit and one barrier a round.  Measured
// (16384^2 with 8- and 4-connectivity, 4096^2 with 4, 512^2 with 8; whole calls one
// after another): 1386, 1367, 252, 117 us; before scans ran in pairs on lines in
// registers, with a barrier of seven round trips and seed strips only: 1520, 1725,
// 324, 146.
#include "iwpp_device.hpp"
#include "iwpp_internal.hpp"

namespace iwpp {
namespace mr {

constexpr int T = kMrTile;     // tile side: lanes map to the 64 columns (or rows)
static_assert(T == 64, "lanes map to tile rows and columns");
constexpr int kRows = T + 2;   // region rows with the halo
constexpr int P = 68;          // LDS row pitch: 17 dwords, so column walks hit distinct banks
constexpr int kOff = 4;        // LDS byte offset of tile column 0 (4-byte aligned chunks)
constexpr int kRegion = kRows * P + 4;  // the last row's column 64 spills into the pad
constexpr int kStageCap = 64;  // LDS work-list stage per wave (iwpp_options.stage_depth caps it)
constexpr uint32_t kMaxRounds = 1u << 20;

__device__ __forceinline__ int lidx(int y, int x) { return (y + 1) * P + x + kOff; }  // y, x in [-1, 64]
// Column 65 of rows -1..64 is never written by a tile load: it is cleared once
// per kernel and read as zeros (it shares bytes with no other column).
constexpr int kZeroCol = T + 1;

struct WaveLds {
  uint8_t J[kRegion];
  uint8_t I[kRegion];
};

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t min_u8x4(uint32_t a, uint32_t b) {
  uint32_t r = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t x = (a >> (8 * k)) & 0xffu, y = (b >> (8 * k)) & 0xffu;
    r |= (x < y ? x : y) << (8 * k);
  }
  return r;
}

__device__ __forceinline__ uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

// A global tile id resolved to its image and tile coordinates (wave-uniform).
struct TileRef {
  MrJob j;
  int ty, tx;
};

__device__ __forceinline__ TileRef tile_ref(const MrArgs& a, uint32_t t) {
  TileRef r;
  r.j = a.job0;
  if (a.njobs != 1u) r.j = uniform(a.jobs[a.tile_job[t]]);
  const uint32_t lt = t - r.j.tile_base;
  r.ty = (int)(lt / (uint32_t)r.j.tiles_x);
  r.tx = (int)(lt - (uint32_t)r.ty * (uint32_t)r.j.tiles_x);
  return r;
}

// Offset that makes a raw buffer access fall outside every buffer (reads 0).
constexpr uint32_t kOutside = 0xFFFFFFF0u;

// Load the (T+2) x (T+2) region of tile (ty, tx) -- the tile and its one-pixel
// halo -- into LDS.  Pixels outside the image read as J = I = 0, which can
// neither raise nor be raised, i.e. they are not neighbours.  In the seed pass
// J is the marker clamped to the mask.  The 66 rows are 264 chunks of 16
// bytes (five per lane) plus 132 halo bytes, each read as the 4-byte word
// that ends at it (three per lane); every load is issued, with no branch in
// between, before the first LDS write, so a visit waits for memory once.
// Loads that would leave the image are pointed outside the buffer (they read
// 0; a raw buffer load that crosses the buffer's end reads 0 as a whole, so
// no load may reach past the image).  A chunk cut by the right edge of the
// image -- one chunk column of the tiles at that edge -- is read byte by byte
// in a second pass.
//
// Seed pass only: with `fresh_top` the halo row above the tile (its 64 bytes,
// not the corners) is read from the output, where the tile above has already
// been written by this wave; a value there is a valid lower bound of the
// result like any other, so it only lets the flood cross the edge earlier.
//
// Propagation rounds (not the seed pass) read the halo columns and corners
// from the neighbouring tiles' border-column blocks (`cols`, `cols_bytes`
// long, rewritten whenever a tile is written): one byte per lane from four
// 64-byte runs instead of 132 words from 66 image rows.
template <bool kSeed>
__device__ void load_region(const TileRef& tr, WaveLds& L, bool fresh_top = false, const uint8_t* cols = nullptr,
                            uint32_t cols_bytes = 0, uint32_t t = 0) {
  const MrJob& a = tr.j;
  const int lv = local_copy(lane());
  const int y0 = tr.ty * T, x0 = tr.tx * T;
  // Buffer resources over the image rows the region touches, [yb, ye): offsets
  // stay 32-bit whatever the image size (a 66-row band of a row of up to 2^31
  // pixels), so images beyond 2^32 pixels are addressed like small ones.
  const int yb = y0 > 0 ? y0 - 1 : 0, ye = y0 + T + 1 < a.h ? y0 + T + 1 : a.h;
  const uint32_t band = (uint32_t)(ye - yb) * (uint32_t)a.w;
  const size_t base = (size_t)yb * (size_t)(uint32_t)a.w;
  const __amdgpu_buffer_rsrc_t rj = make_rsrc((kSeed ? a.marker : a.out) + base, band);
  const __amdgpu_buffer_rsrc_t ri = make_rsrc(a.mask + base, band);
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(a.out + base, band);
  const int rem = a.w - x0;  // image columns from this tile's first column on
  const int cp = (rem < T && (rem & 15) != 0) ? rem >> 4 : -1;  // the cut chunk column, if any
  constexpr int kMain = kRows * 4, kHalo = kRows * 2;
  constexpr int kPerMain = (kMain + kWave - 1) / kWave, kPerHalo = (kHalo + kWave - 1) / kWave;
  v4u vj[kPerMain], vi[kPerMain];
  uint32_t hj[kPerHalo], hi[kPerHalo];
  uint32_t xm[kPerMain], xh[kPerHalo];  // complement of what was read inside the image (erosion), else 0
#pragma unroll
  for (int k = 0; k < kPerMain; ++k) {
    const int idx = lv + k * kWave;
    const int c = idx & 3;
    const int y = y0 - 1 + (idx >> 2), xs = x0 + 16 * c;
    const bool ok = idx < kMain && y >= 0 && y < a.h && xs + 16 <= a.w;
    xm[k] = ok ? a.inv : 0u;
    const uint32_t off = ok ? (uint32_t)(y - yb) * (uint32_t)a.w + (uint32_t)xs : kOutside;
    vj[k] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rj, off, 0, kSc1));
    vi[k] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(ri, off, 0, kSc1));
  }
  v4u vtop = {0u, 0u, 0u, 0u};
  if (kSeed && fresh_top) {  // wave-uniform; lanes 0..3 hold the row above
    const int y = y0 - 1, xs = x0 + 16 * (lv & 3);
    const bool ok = lv < 4 && y >= 0 && xs + 16 <= a.w;
    const uint32_t off = ok ? (uint32_t)(y - yb) * (uint32_t)a.w + (uint32_t)xs : kOutside;
    vtop = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(ro, off, 0, kSc1));
    // lanes 0..3 load the same chunks as vj[0] (row y0 - 1), so xm[0] applies
    if (lv < 4) vj[0] = vtop;
  }
  if (kSeed) {
#pragma unroll
    for (int k = 0; k < kPerHalo; ++k) {
      const int idx = lv + k * kWave;
      const int y = y0 - 1 + (idx >> 1);
      const int x = (idx & 1) ? x0 + T : x0 - 1;
      const bool ok = idx < kHalo && y >= 0 && y < a.h && x >= 3 && x < a.w;
      xh[k] = ok ? a.inv : 0u;
      const uint32_t off = ok ? (uint32_t)(y - yb) * (uint32_t)a.w + (uint32_t)(x - 3) : kOutside;
      hj[k] = __builtin_amdgcn_raw_buffer_load_b32(rj, off, 0, kSc1);
      hi[k] = __builtin_amdgcn_raw_buffer_load_b32(ri, off, 0, kSc1);
    }
  } else {
    // Lane l: row l of the left neighbour's right column and of the right
    // neighbour's left column (J and I); lanes 0..3 also one corner each:
    // top-left, top-right, bottom-left, bottom-right.
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(cols, cols_bytes);
    const int l = local_copy(lane());
    const int tx_n = tr.j.tiles_x, ty_n = tr.j.tiles_y;
    const bool has_l = tr.tx > 0, has_r = tr.tx + 1 < tx_n;
    const uint32_t bl = (t - 1u) * 256u, br = (t + 1u) * 256u;
    const uint32_t ol = has_l ? bl + 64u + (uint32_t)l : kOutside, or_ = has_r ? br + (uint32_t)l : kOutside;
    hj[0] = __builtin_amdgcn_raw_buffer_load_b8(rc, ol, 0, kSc1);
    hi[0] = __builtin_amdgcn_raw_buffer_load_b8(rc, ol == kOutside ? kOutside : ol + 128u, 0, kSc1);
    hj[1] = __builtin_amdgcn_raw_buffer_load_b8(rc, or_, 0, kSc1);
    hi[1] = __builtin_amdgcn_raw_buffer_load_b8(rc, or_ == kOutside ? kOutside : or_ + 128u, 0, kSc1);
    const int cdy = (l & 2) ? 1 : -1, cdx = (l & 1) ? 1 : -1;
    const bool has_c = l < 4 && tr.ty + cdy >= 0 && tr.ty + cdy < ty_n && tr.tx + cdx >= 0 && tr.tx + cdx < tx_n;
    // the corner pixel is the diagonal tile's (right column if it lies left) row 63 (if above) or 0
    const uint32_t tc = (uint32_t)((int)t + cdy * tx_n + cdx);
    const uint32_t oc = has_c ? tc * 256u + (cdx < 0 ? 64u : 0u) + (cdy < 0 ? 63u : 0u) : kOutside;
    hj[2] = __builtin_amdgcn_raw_buffer_load_b8(rc, oc, 0, kSc1);
    hi[2] = __builtin_amdgcn_raw_buffer_load_b8(rc, oc == kOutside ? kOutside : oc + 128u, 0, kSc1);
  }
#pragma unroll
  for (int k = 0; k < kPerMain; ++k) {
    const int idx = lv + k * kWave;
    if (idx >= kMain) continue;
    const int ry = idx >> 2, c = idx & 3;
    uint32_t* dj = reinterpret_cast<uint32_t*>(&L.J[lidx(ry - 1, c * 16)]);
    uint32_t* di = reinterpret_cast<uint32_t*>(&L.I[lidx(ry - 1, c * 16)]);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      dj[d] = kSeed ? min_u8x4(vj[k][d] ^ xm[k], vi[k][d] ^ xm[k]) : vj[k][d] ^ xm[k];
      di[d] = vi[k][d] ^ xm[k];
    }
  }
  if (kSeed) {
#pragma unroll
    for (int k = 0; k < kPerHalo; ++k) {
      const int idx = lv + k * kWave;
      if (idx >= kHalo) continue;
      const int ry = idx >> 1;
      const uint32_t jb = (hj[k] ^ xh[k]) >> 24, ib = (hi[k] ^ xh[k]) >> 24;
      const int at = lidx(ry - 1, (idx & 1) ? T : -1);
      L.J[at] = (uint8_t)umin(jb, ib);
      L.I[at] = (uint8_t)ib;
    }
  } else {
    const int l = local_copy(lane());
    L.J[lidx(l, -1)] = (uint8_t)hj[0];
    L.I[lidx(l, -1)] = (uint8_t)hi[0];
    L.J[lidx(l, T)] = (uint8_t)hj[1];
    L.I[lidx(l, T)] = (uint8_t)hi[1];
    if (l < 4) {
      const int at = lidx((l & 2) ? T : -1, (l & 1) ? T : -1);
      L.J[at] = (uint8_t)hj[2];
      L.I[at] = (uint8_t)hi[2];
    }
  }
  if (cp >= 0) {  // wave-uniform: only tiles cut by the right edge of the image
    const int nb = rem - 16 * cp, xs = x0 + 16 * cp;
#pragma unroll
    for (int k = 0; k < (kRows + kWave - 1) / kWave; ++k) {
      const int ry = lv + k * kWave;
      const int y = y0 - 1 + ry;
      const bool row_ok = ry < kRows && y >= 0 && y < a.h;
      uint32_t bj[15], bi[15];
      const uint32_t xb = row_ok ? a.inv & 0xffu : 0u;
#pragma unroll
      for (int b = 0; b < 15; ++b) {
        const uint32_t off = (row_ok && b < nb) ? (uint32_t)(y - yb) * (uint32_t)a.w + (uint32_t)(xs + b) : kOutside;
        bj[b] = __builtin_amdgcn_raw_buffer_load_b8(rj, off, 0, kSc1) ^ xb;
        bi[b] = __builtin_amdgcn_raw_buffer_load_b8(ri, off, 0, kSc1) ^ xb;
      }
      if (ry < kRows) {
#pragma unroll
        for (int b = 0; b < 15; ++b) {
          if (b >= nb) continue;  // (a break would put the bytes in scratch)
          const int at = lidx(ry - 1, 16 * cp + b);
          L.J[at] = (uint8_t)(kSeed ? umin(bj[b], bi[b]) : bj[b]);
          L.I[at] = (uint8_t)bi[b];
        }
      }
    }
  }
  wave_sync();
}

// Propagation visits load a tile in two parts, so that a listed tile that
// turns out to need no work costs a small fraction of a full load.
//
// The frame: everything the skip test (`border_raisable`) and the border
// marks read -- rows -1, 0, 63 and 64 of the region (J and I, one byte per
// lane and row from the image), the tile's own border columns 0 and 63 and
// the halo columns -1 and 64 (J and I, from the border-column blocks of the
// tile and of its left and right neighbours), and the four halo corners
// (from the diagonal neighbours' blocks).  Rows and columns outside the image
// read as 0.
__device__ void load_frame(const TileRef& tr, WaveLds& L, const uint8_t* cols, uint32_t cols_bytes, uint32_t t) {
  const MrJob& a = tr.j;
  const int y0 = tr.ty * T, x0 = tr.tx * T, l = local_copy(lane());
  const int yb = y0 > 0 ? y0 - 1 : 0, ye = y0 + T + 1 < a.h ? y0 + T + 1 : a.h;
  const uint32_t band = (uint32_t)(ye - yb) * (uint32_t)a.w;
  const size_t base = (size_t)yb * (size_t)(uint32_t)a.w;
  const __amdgpu_buffer_rsrc_t ro = make_rsrc(a.out + base, band);
  const __amdgpu_buffer_rsrc_t ri = make_rsrc(a.mask + base, band);
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(cols, cols_bytes);
  constexpr int kFrameRows[4] = {-1, 0, T - 1, T};
  uint32_t fj[4], fi[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int y = y0 + kFrameRows[k], x = x0 + l;
    const bool ok = y >= 0 && y < a.h && x < a.w;
    const uint32_t off = ok ? (uint32_t)(y - yb) * (uint32_t)a.w + (uint32_t)x : kOutside;
    const uint32_t xb = ok ? a.inv & 0xffu : 0u;
    fj[k] = __builtin_amdgcn_raw_buffer_load_b8(ro, off, 0, kSc1) ^ xb;
    fi[k] = __builtin_amdgcn_raw_buffer_load_b8(ri, off, 0, kSc1) ^ xb;
  }
  // Columns: own block [J left | J right | I left | I right], the left
  // neighbour's right column, the right neighbour's left column (lane = row).
  const uint32_t bo = t * 256u;
  const uint32_t oj0 = __builtin_amdgcn_raw_buffer_load_b8(rc, bo + (uint32_t)l, 0, kSc1);
  const uint32_t oj1 = __builtin_amdgcn_raw_buffer_load_b8(rc, bo + 64u + (uint32_t)l, 0, kSc1);
  const uint32_t oi0 = __builtin_amdgcn_raw_buffer_load_b8(rc, bo + 128u + (uint32_t)l, 0, kSc1);
  const uint32_t oi1 = __builtin_amdgcn_raw_buffer_load_b8(rc, bo + 192u + (uint32_t)l, 0, kSc1);
  const int tx_n = tr.j.tiles_x, ty_n = tr.j.tiles_y;
  const bool has_l = tr.tx > 0, has_r = tr.tx + 1 < tx_n;
  const uint32_t ol = has_l ? (t - 1u) * 256u + 64u + (uint32_t)l : kOutside;
  const uint32_t or_ = has_r ? (t + 1u) * 256u + (uint32_t)l : kOutside;
  const uint32_t hjl = __builtin_amdgcn_raw_buffer_load_b8(rc, ol, 0, kSc1);
  const uint32_t hil = __builtin_amdgcn_raw_buffer_load_b8(rc, ol == kOutside ? kOutside : ol + 128u, 0, kSc1);
  const uint32_t hjr = __builtin_amdgcn_raw_buffer_load_b8(rc, or_, 0, kSc1);
  const uint32_t hir = __builtin_amdgcn_raw_buffer_load_b8(rc, or_ == kOutside ? kOutside : or_ + 128u, 0, kSc1);
  // Corners, lanes 0..3: top-left, top-right, bottom-left, bottom-right.
  const int cdy = (l & 2) ? 1 : -1, cdx = (l & 1) ? 1 : -1;
  const bool has_c = l < 4 && tr.ty + cdy >= 0 && tr.ty + cdy < ty_n && tr.tx + cdx >= 0 && tr.tx + cdx < tx_n;
  const uint32_t tc = (uint32_t)((int)t + cdy * tx_n + cdx);
  const uint32_t oc = has_c ? tc * 256u + (cdx < 0 ? 64u : 0u) + (cdy < 0 ? 63u : 0u) : kOutside;
  const uint32_t cj = __builtin_amdgcn_raw_buffer_load_b8(rc, oc, 0, kSc1);
  const uint32_t ci = __builtin_amdgcn_raw_buffer_load_b8(rc, oc == kOutside ? kOutside : oc + 128u, 0, kSc1);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    L.J[lidx(kFrameRows[k], l)] = (uint8_t)fj[k];
    L.I[lidx(kFrameRows[k], l)] = (uint8_t)fi[k];
  }
  L.J[lidx(l, 0)] = (uint8_t)oj0;
  L.J[lidx(l, T - 1)] = (uint8_t)oj1;
  L.I[lidx(l, 0)] = (uint8_t)oi0;
  L.I[lidx(l, T - 1)] = (uint8_t)oi1;
  L.J[lidx(l, -1)] = (uint8_t)hjl;
  L.I[lidx(l, -1)] = (uint8_t)hil;
  L.J[lidx(l, T)] = (uint8_t)hjr;
  L.I[lidx(l, T)] = (uint8_t)hir;
  if (l < 4) {
    const int at = lidx((l & 2) ? T : -1, (l & 1) ? T : -1);
    L.J[at] = (uint8_t)cj;
    L.I[at] = (uint8_t)ci;
  }
  wave_sync();
}

// The rest of a propagation visit's region: rows 1..62 of the tile (J and I),
// as 16-byte chunks (four per row), and byte by byte where a chunk is cut by
// the image's right edge (see load_region).
__device__ void load_interior(const TileRef& tr, WaveLds& L) {
  const MrJob& a = tr.j;
  const int lv = local_copy(lane());
  const int y0 = tr.ty * T, x0 = tr.tx * T;
  const int yb = y0 > 0 ? y0 - 1 : 0, ye = y0 + T + 1 < a.h ? y0 + T + 1 : a.h;
  const uint32_t band = (uint32_t)(ye - yb) * (uint32_t)a.w;
  const size_t base = (size_t)yb * (size_t)(uint32_t)a.w;
  const __amdgpu_buffer_rsrc_t rj = make_rsrc(a.out + base, band);
  const __amdgpu_buffer_rsrc_t ri = make_rsrc(a.mask + base, band);
  const int rem = a.w - x0;
  const int cp = (rem < T && (rem & 15) != 0) ? rem >> 4 : -1;
  constexpr int kChunks = (T - 2) * 4;
  constexpr int kPer = (kChunks + kWave - 1) / kWave;
  v4u vj[kPer], vi[kPer];
  uint32_t xm[kPer];  // complement of what was read inside the image (erosion), else 0
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int idx = lv + k * kWave;
    const int c = idx & 3;
    const int y = y0 + 1 + (idx >> 2), xs = x0 + 16 * c;
    const bool ok = idx < kChunks && y < a.h && xs + 16 <= a.w;
    xm[k] = ok ? a.inv : 0u;
    const uint32_t off = ok ? (uint32_t)(y - yb) * (uint32_t)a.w + (uint32_t)xs : kOutside;
    vj[k] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rj, off, 0, kSc1));
    vi[k] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(ri, off, 0, kSc1));
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int idx = lv + k * kWave;
    if (idx >= kChunks) continue;
    const int ry = 1 + (idx >> 2), c = idx & 3;
    uint32_t* dj = reinterpret_cast<uint32_t*>(&L.J[lidx(ry, c * 16)]);
    uint32_t* di = reinterpret_cast<uint32_t*>(&L.I[lidx(ry, c * 16)]);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      dj[d] = vj[k][d] ^ xm[k];
      di[d] = vi[k][d] ^ xm[k];
    }
  }
  if (cp >= 0) {  // wave-uniform: only tiles cut by the right edge of the image
    const int nb = rem - 16 * cp, xs = x0 + 16 * cp;
    const int ry = 1 + lv;
    const int y = y0 + ry;
    const bool row_ok = ry < T - 1 && y < a.h;
    uint32_t bj[15], bi[15];
    const uint32_t xb = row_ok ? a.inv & 0xffu : 0u;
#pragma unroll
    for (int b = 0; b < 15; ++b) {
      const uint32_t off = (row_ok && b < nb) ? (uint32_t)(y - yb) * (uint32_t)a.w + (uint32_t)(xs + b) : kOutside;
      bj[b] = __builtin_amdgcn_raw_buffer_load_b8(rj, off, 0, kSc1) ^ xb;
      bi[b] = __builtin_amdgcn_raw_buffer_load_b8(ri, off, 0, kSc1) ^ xb;
    }
    if (ry < T - 1) {
#pragma unroll
      for (int b = 0; b < 15; ++b) {
        if (b >= nb) continue;  // (a break would put the bytes in scratch)
        const int at = lidx(ry, 16 * cp + b);
        L.J[at] = (uint8_t)bj[b];
        L.I[at] = (uint8_t)bi[b];
      }
    }
  }
  wave_sync();
}

// Write the tile interior back to the image (device-coherent stores).
__device__ void store_tile(const TileRef& tr, const WaveLds& L) {
  const MrJob& a = tr.j;
  const int y0 = tr.ty * T, x0 = tr.tx * T;
  const int ye = y0 + T < a.h ? y0 + T : a.h;  // the tile's rows, as a band of their own (see load_region)
  const __amdgpu_buffer_rsrc_t ro =
      make_rsrc(a.out + (size_t)y0 * (size_t)(uint32_t)a.w, (uint32_t)(ye - y0) * (uint32_t)a.w);
  for (int idx = local_copy(lane()); idx < T * 4; idx += kWave) {
    const int ry = idx >> 2, c = idx & 3;
    const int y = y0 + ry, xs = x0 + c * 16;
    if (y >= a.h || xs >= a.w) continue;
    const uint32_t* s = reinterpret_cast<const uint32_t*>(&L.J[lidx(ry, c * 16)]);
    v4u v = {s[0] ^ a.inv, s[1] ^ a.inv, s[2] ^ a.inv, s[3] ^ a.inv};
    const uint32_t off = (uint32_t)ry * (uint32_t)a.w + (uint32_t)xs;
    if (xs + 16 <= a.w) {
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v), ro, off, 0, kSc1);
    } else {
      const int nb = a.w - xs;
#pragma unroll
      for (int b = 0; b < 16; ++b)
        if (b < nb)
          __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(v[b >> 2] >> (8 * (b & 3))), ro, off + b, 0, kSc1);
    }
  }
}

// Write the tile's border columns (J, and with `mask` also I) into its block
// of `cols`: [J left | J right | I left | I right], 64 bytes each.
__device__ void store_cols(const MrArgs& a, uint32_t t, const WaveLds& L, bool mask) {
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(a.cols + (size_t)t * 256u, 256u);
  const int l = local_copy(lane());
  __builtin_amdgcn_raw_buffer_store_b8(L.J[lidx(l, 0)], rc, (uint32_t)l, 0, kSc1);
  __builtin_amdgcn_raw_buffer_store_b8(L.J[lidx(l, T - 1)], rc, 64u + (uint32_t)l, 0, kSc1);
  if (mask) {
    __builtin_amdgcn_raw_buffer_store_b8(L.I[lidx(l, 0)], rc, 128u + (uint32_t)l, 0, kSc1);
    __builtin_amdgcn_raw_buffer_store_b8(L.I[lidx(l, T - 1)], rc, 192u + (uint32_t)l, 0, kSc1);
  }
}

// Rows and columns of the tile that changed since the scans that could carry
// the change further last ran (bit = row or column index, wave-uniform).  After
// a scan in direction D every pixel dominates the offers of its D-predecessors
// (the pixel before it along D: left for rows forward, right for rows backward,
// the row above -- three pixels with 8-connectivity -- for columns forward, the
// row below for columns backward), and it keeps dominating them until one of
// those predecessors rises.  So a scan only needs the 16-wide chunks whose
// predecessors changed since it last ran, plus any chunk after one that it has
// just changed; and the tile is locally stable exactly when all sets are empty
// (the four scans' predecessors are all eight neighbours, or all four).
//
// Along a line of its own (rows; columns with 4-connectivity) a scan in one
// direction leaves intact what the other has reached: with x dominating its
// left offers and x' the result of the backward scan, x'[k-1] <= max(x[k-1],
// x'[k]), so min(x'[k-1], I[k]) <= max(x[k], x'[k]) = x'[k].  So rows need one
// set for both directions, and a scan never adds to its own axis' set.  With
// 8-connectivity a column scan's changes do reach the other direction, through
// the diagonals.
struct Dirty {
  uint64_t r_cf, r_cb;  // rows changed since the last column scan forward / backward
  uint64_t c_r;         // columns changed since the last row scans
  __device__ bool empty() const { return (r_cf | r_cb | c_r) == 0ull; }
};

// Apply every halo pixel's offer to the border pixels it touches, once:
// J(p) <- max(J(p), min(J(h), I(p))) for border pixel p and halo neighbour h.
// Halo pixels do not change during a visit and J only rises, so afterwards no
// halo offer can raise anything again and the scans can ignore the halo (it
// acts as zeros there).  Rows first, then columns, so a corner pixel takes
// both.  Sets the rows and the columns that hold a border pixel that rose.
template <int CONN>
__device__ void fold_halo(WaveLds& L, uint64_t& rows, uint64_t& cols) {
  const int l = local_copy(lane());
  auto offer = [&](int hy0, int hx0, int hy1, int hx1, int hy2, int hx2) {  // max of the halo neighbours
    uint32_t h = L.J[lidx(hy1, hx1)];
    if (CONN == 8) h = umax(h, umax((uint32_t)L.J[lidx(hy0, hx0)], (uint32_t)L.J[lidx(hy2, hx2)]));
    return h;
  };
  const uint32_t ht = offer(-1, l - 1, -1, l, -1, l + 1), hb = offer(T, l - 1, T, l, T, l + 1);
  const uint32_t jt = L.J[lidx(0, l)], it = L.I[lidx(0, l)], jb = L.J[lidx(T - 1, l)], ib = L.I[lidx(T - 1, l)];
  const uint32_t nt = umax(jt, umin(ht, it)), nb = umax(jb, umin(hb, ib));
  L.J[lidx(0, l)] = (uint8_t)nt;
  L.J[lidx(T - 1, l)] = (uint8_t)nb;
  const uint64_t top = ballot(nt != jt), bot = ballot(nb != jb);  // lane = column
  // The column phase reads corners that other lanes wrote in the row phase
  // (lane 63 wrote (0, 63), lane 0 wrote (63, 0)): order the two phases.
  wave_sync();
  const uint32_t hl = offer(l - 1, -1, l, -1, l + 1, -1), hr = offer(l - 1, T, l, T, l + 1, T);
  const uint32_t jl = L.J[lidx(l, 0)], il = L.I[lidx(l, 0)], jr = L.J[lidx(l, T - 1)], ir = L.I[lidx(l, T - 1)];
  const uint32_t nl = umax(jl, umin(hl, il)), nr = umax(jr, umin(hr, ir));
  L.J[lidx(l, 0)] = (uint8_t)nl;
  L.J[lidx(l, T - 1)] = (uint8_t)nr;
  const uint64_t left = ballot(nl != jl), right = ballot(nr != jr);  // lane = row
  wave_sync();
  rows = left | right | (top ? 1ull : 0ull) | (bot ? 1ull << (T - 1) : 0ull);
  cols = top | bot | (left ? 1ull : 0ull) | (right ? 1ull << (T - 1) : 0ull);
}

// The two scans of an axis of the tile in LDS, after `fold_halo`: the halo is
// ignored.  Vertical scans walk the rows with lane = column, using the previous
// row's values of the three (8-conn) or one (4-conn) upper/lower neighbours;
// horizontal scans walk the columns with lane = row, using the previous column.
//
// A scan is a serial chain -- every step waits for the one before -- of two to
// five instructions a step, and one wave has 64 of them; four waves per SIMD do
// not cover the wait.  So the forward and the backward scan of an axis run
// together, in four passes of one 16-wide chunk each: the forward scan takes
// chunks 0, 1, 2, 3, the backward scan 3, 2, 1, 0, never the same chunk in one
// pass, and their independent steps fill each other's waits.  Each works on what
// the other has raised.  Every value is a valid update of the ones it was
// computed from and at least what either scan alone would give, and on a line
// the limit is the larger of the two scans, so after a pair the line is stable.
//
// The lane's whole line stays in registers over both scans (rows packed, 16
// words and 16 of mask; columns a register a pixel): it is read from LDS once,
// not once a scan, all of it before the first step with 4-connectivity, and by
// chunk as scans need it with 8.  Of a chunk whose predecessors did not change
// since a scan last ran (`Dirty`), and that follows no chunk the scan changed,
// the scan is skipped; a chunk that no scan changed is not written back.
//
// Measured (us, one scan at a time from LDS -> pairs from LDS -> pairs in
// registers): 16384^2 with 4-connectivity 1728, 1707, 1635; 4096^2 352, 342,
// 331; with 8-connectivity, where only row scans pair, 16384^2 1551, 1537, 1530.
constexpr int kChunk = 16;
static_assert(T == 4 * kChunk, "four chunks per scan: with an even number no pass has both scans on one chunk");

// Predecessor lines of chunk [x0, x0 + 16) in the scan's direction.
__device__ __forceinline__ uint64_t chunk_preds(int x0, bool forward) {
  const uint64_t w = 0xFFFFull << x0;
  return forward ? w >> 1 : w << 1;
}

// d | (a ^ b): collects whether anything changed, one instruction a step.
__device__ __forceinline__ uint32_t or_diff(uint32_t a, uint32_t b, uint32_t d) {
  asm("v_bitop3_b32 %0, %1, %2, %0 bitop3:0xbe" : "+v"(d) : "v"(a), "v"(b));
  return d;
}

// Row scans (lane = row) on packed words: one step is a byte-selecting max of
// the old pixel and the previous result, then a byte-selecting min with the
// mask written into the pixel's byte in place (SDWA with the other bytes
// preserved), two instructions per pixel with no unpacking or repacking.
// MR_HSTEP: pixel byte K of word W, previous result in byte PK of word PW.
// MR_HSTEP2: such a step of each scan, alternating (the instruction between
// also is the wait state that reading a just-written byte needs).
#define MR_HSTEP(W, PW, I, K, PK)                                                                       \
  do {                                                                                                  \
    uint32_t m_;                                                                                        \
    asm("v_max_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #K              \
        " src1_sel:BYTE_" #PK                                                                           \
        : "=v"(m_)                                                                                      \
        : "v"(W), "v"(PW));                                                                             \
    asm("v_min_u32_sdwa %0, %1, %2 dst_sel:BYTE_" #K " dst_unused:UNUSED_PRESERVE src0_sel:DWORD"      \
        " src1_sel:BYTE_" #K                                                                            \
        : "+v"(W)                                                                                       \
        : "v"(m_), "v"(I));                                                                             \
  } while (0)
#define MR_HSTEP2(W, PW, I, K, PK, W2, PW2, I2, K2, PK2)                                                \
  do {                                                                                                  \
    uint32_t m_, m2_;                                                                                   \
    asm("v_max_u32_sdwa %0, %2, %4 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #K              \
        " src1_sel:BYTE_" #PK "\n\t"                                                                    \
        "v_max_u32_sdwa %1, %3, %5 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #K2             \
        " src1_sel:BYTE_" #PK2 "\n\t"                                                                   \
        "v_min_u32_sdwa %2, %0, %6 dst_sel:BYTE_" #K " dst_unused:UNUSED_PRESERVE src0_sel:DWORD"      \
        " src1_sel:BYTE_" #K "\n\t"                                                                     \
        "v_min_u32_sdwa %3, %1, %7 dst_sel:BYTE_" #K2 " dst_unused:UNUSED_PRESERVE src0_sel:DWORD"     \
        " src1_sel:BYTE_" #K2                                                                           \
        : "=&v"(m_), "=&v"(m2_), "+&v"(W), "+&v"(W2)                                                      \
        : "v"(PW), "v"(PW2), "v"(I), "v"(I2));                                                          \
  } while (0)

// MR_HSTEP1: MR_HSTEP2 with the previous results in the same words.
#define MR_HSTEP1(W, I, K, PK, W2, I2, K2, PK2)                                                         \
  do {                                                                                                  \
    uint32_t m_, m2_;                                                                                   \
    asm("v_max_u32_sdwa %0, %2, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #K              \
        " src1_sel:BYTE_" #PK "\n\t"                                                                    \
        "v_max_u32_sdwa %1, %3, %3 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_" #K2             \
        " src1_sel:BYTE_" #PK2 "\n\t"                                                                   \
        "v_min_u32_sdwa %2, %0, %4 dst_sel:BYTE_" #K " dst_unused:UNUSED_PRESERVE src0_sel:DWORD"      \
        " src1_sel:BYTE_" #K "\n\t"                                                                     \
        "v_min_u32_sdwa %3, %1, %5 dst_sel:BYTE_" #K2 " dst_unused:UNUSED_PRESERVE src0_sel:DWORD"     \
        " src1_sel:BYTE_" #K2                                                                           \
        : "=&v"(m_), "=&v"(m2_), "+&v"(W), "+&v"(W2)                                                      \
        : "v"(I), "v"(I2));                                                                             \
  } while (0)

// One pass of the row scans on the row in registers: the forward scan (kF) on
// words [4 C, 4 C + 4), the backward scan (kB) on the mirrored chunk.  What
// precedes a chunk is in the word beside it, whatever has been skipped.
template <int C, bool kF, bool kB>
__device__ __forceinline__ void row_pass(uint32_t (&w)[T / 4], const uint32_t (&m)[T / 4], uint32_t& df, uint32_t& db) {
  const uint32_t zero = 0u;  // before the first pixel: the halo acts as zeros
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int d = 4 * C + k, e = T / 4 - 1 - d;
    const uint32_t of = w[d], ob = w[e];
    const uint32_t pf = d > 0 ? w[d > 0 ? d - 1 : 0] : zero, pb = d > 0 ? w[d > 0 ? e + 1 : e] : zero;
    if (kF && kB) {
      MR_HSTEP2(w[d], pf, m[d], 0, 3, w[e], pb, m[e], 3, 0);
      MR_HSTEP1(w[d], m[d], 1, 0, w[e], m[e], 2, 3);
      MR_HSTEP1(w[d], m[d], 2, 1, w[e], m[e], 1, 2);
      MR_HSTEP1(w[d], m[d], 3, 2, w[e], m[e], 0, 1);
    } else if (kF) {
      MR_HSTEP(w[d], pf, m[d], 0, 3);
      MR_HSTEP(w[d], w[d], m[d], 1, 0);
      MR_HSTEP(w[d], w[d], m[d], 2, 1);
      MR_HSTEP(w[d], w[d], m[d], 3, 2);
    } else {
      MR_HSTEP(w[e], pb, m[e], 3, 0);
      MR_HSTEP(w[e], w[e], m[e], 2, 3);
      MR_HSTEP(w[e], w[e], m[e], 1, 2);
      MR_HSTEP(w[e], w[e], m[e], 0, 1);
    }
    if (kF) df = or_diff(of, w[d], df);
    if (kB) db = or_diff(ob, w[e], db);
  }
}

// The lane's row in registers, chunk by chunk as scans need them (bit c of
// `have`); bit c of `changed`: to be written back.
struct Row {
  uint32_t w[T / 4], m[T / 4];
  uint32_t have = 0u, changed = 0u;
};

template <int C>
__device__ __forceinline__ void load_row_chunk(const uint32_t* jp, const uint32_t* ip, Row& r) {
#pragma unroll
  for (int d = 4 * C; d < 4 * C + 4; ++d) {
    r.w[d] = jp[d];
    r.m[d] = ip[d];
  }
}

// A pass with its chunks' needs; returns the rows that changed.
template <int C, bool kDirty>
__device__ __forceinline__ uint64_t row_chunks(const uint32_t* jp, const uint32_t* ip, Row& r, uint64_t dirty, bool& f, bool& b) {
  constexpr int cf = C, cb = T / kChunk - 1 - C;
  uint32_t df = 0, db = 0;
  if (!kDirty) {
    row_pass<C, true, true>(r.w, r.m, df, db);
  } else {
    f = f || (dirty & chunk_preds(cf * kChunk, true)) != 0ull;
    b = b || (dirty & chunk_preds(cb * kChunk, false)) != 0ull;
    // The chunk, if the other scan has not loaded it, and the word before it.
    if (f && !(r.have >> cf & 1u)) load_row_chunk<cf>(jp, ip, r);
    if (b && !(r.have >> cb & 1u)) load_row_chunk<cb>(jp, ip, r);
    r.have |= (f ? 1u << cf : 0u) | (b ? 1u << cb : 0u);
    if (C > 0 && f && !(r.have >> (C > 0 ? cf - 1 : 0) & 1u)) r.w[C > 0 ? 4 * cf - 1 : 0] = jp[4 * cf - 1];
    if (C > 0 && b && !(r.have >> (C > 0 ? cb + 1 : 0) & 1u)) r.w[C > 0 ? 4 * cb + 4 : 0] = jp[4 * cb + 4];
    if (f && b)
      row_pass<C, true, true>(r.w, r.m, df, db);
    else if (f)
      row_pass<C, true, false>(r.w, r.m, df, db);
    else if (b)
      row_pass<C, false, true>(r.w, r.m, df, db);
  }
  const uint64_t rf = ballot(df != 0u), rb = ballot(db != 0u);
  f = rf != 0ull;
  b = rb != 0ull;
  r.changed |= (f ? 1u << cf : 0u) | (b ? 1u << cb : 0u);
  return rf | rb;
}

// Both row scans (lane = row); returns the rows that changed.
template <bool kDirty>
__device__ __forceinline__ uint64_t row_pair(WaveLds& L, int l, uint64_t dirty) {
  uint32_t* jp = reinterpret_cast<uint32_t*>(&L.J[lidx(l, 0)]);
  const uint32_t* ip = reinterpret_cast<const uint32_t*>(&L.I[lidx(l, 0)]);
  Row r;
  if (!kDirty) {
    load_row_chunk<0>(jp, ip, r);
    load_row_chunk<3>(jp, ip, r);
    load_row_chunk<1>(jp, ip, r);
    load_row_chunk<2>(jp, ip, r);
  }
  bool f = false, b = false;
  uint64_t rows = row_chunks<0, kDirty>(jp, ip, r, dirty, f, b);
  rows |= row_chunks<1, kDirty>(jp, ip, r, dirty, f, b);
  rows |= row_chunks<2, kDirty>(jp, ip, r, dirty, f, b);
  rows |= row_chunks<3, kDirty>(jp, ip, r, dirty, f, b);
#pragma unroll
  for (int c = 0; c < T / kChunk; ++c) {
    if (r.changed >> c & 1u) {  // a chunk that changed nothing is not written back
#pragma unroll
      for (int d = 4 * c; d < 4 * c + 4; ++d) jp[d] = r.w[d];
    }
  }
  wave_sync();
  return rows;
}
#undef MR_HSTEP
#undef MR_HSTEP1
#undef MR_HSTEP2

// The tile's mask column of this lane, four rows per word (row 4w + b in byte
// b of ic[w]): the mask does not change during a visit, so the column scans
// take it from registers and read only J from LDS.
__device__ __forceinline__ void load_mask_column(const WaveLds& L, uint32_t (&ic)[T / 4]) {
  const int l = local_copy(lane());
#pragma unroll
  for (int w = 0; w < T / 4; ++w) {
    const uint32_t b0 = L.I[lidx(4 * w, l)], b1 = L.I[lidx(4 * w + 1, l)], b2 = L.I[lidx(4 * w + 2, l)],
                   b3 = L.I[lidx(4 * w + 3, l)];
    ic[w] = b0 | (b1 << 8) | (b2 << 16) | (b3 << 24);
  }
}

// One step of the column scans: old values V, previous row's results P, the row's
// mask in byte B of M; the new value goes to N.  J <= I throughout, so
// min(max(J, offers), I) is the update.  With 8-connectivity the two lane shifts
// of the diagonal offers are fused into the max (DPP with zero fill); a DPP read
// of a just-written register needs two wait states, so a step begins with
// collecting the previous step's changes (P against its old value O, into D).
// `column_step2` is a step of each scan, alternating.
#define MR_MIN(D, S, I, B) "v_min_u32_sdwa " D ", " S ", " I " dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_" B "\n\t"
#define MR_DIFF(D, N, V) "v_bitop3_b32 " D ", " N ", " V ", " D " bitop3:0xbe\n\t"
#define MR_SHR(D, P, V) "v_max_u32_dpp " D ", " P ", " V " wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define MR_SHL(D, P, V) "v_max_u32_dpp " D ", " P ", " V " wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define MR_MAX(D, A, B) "v_max_u32 " D ", " A ", " B "\n\t"

template <int CONN, int B>
__device__ __forceinline__ void column_step2(uint32_t& vf, uint32_t& pf, uint32_t& of, uint32_t& df, uint32_t mf,
                                             uint32_t& vb, uint32_t& pb, uint32_t& ob, uint32_t& db, uint32_t mb) {
  uint32_t nf, nb, tf, tb;
#define MR_STEP8(BF, BB)                                                                                            \
  asm(MR_DIFF("%4", "%6", "%12") MR_DIFF("%5", "%7", "%13") MR_SHR("%0", "%6", "%8") MR_SHR("%1", "%7", "%9")         \
          MR_SHL("%2", "%6", "%6") MR_SHL("%3", "%7", "%7") MR_MAX("%0", "%0", "%2") MR_MAX("%1", "%1", "%3")         \
              MR_MIN("%0", "%0", "%10", BF) MR_MIN("%1", "%1", "%11", BB)                                             \
      : "=&v"(nf), "=&v"(nb), "=&v"(tf), "=&v"(tb), "+v"(df), "+v"(db)                                                \
      : "v"(pf), "v"(pb), "v"(vf), "v"(vb), "v"(mf), "v"(mb), "v"(of), "v"(ob))
#define MR_STEP4(BF, BB)                                                                                             \
  asm(MR_DIFF("%2", "%4", "%10") MR_DIFF("%3", "%5", "%11") MR_MAX("%0", "%4", "%6") MR_MAX("%1", "%5", "%7")          \
          MR_MIN("%0", "%0", "%8", BF) MR_MIN("%1", "%1", "%9", BB)                                                    \
      : "=&v"(nf), "=&v"(nb), "+v"(df), "+v"(db)                                                                       \
      : "v"(pf), "v"(pb), "v"(vf), "v"(vb), "v"(mf), "v"(mb), "v"(of), "v"(ob))
  if constexpr (CONN == 8) {
    if constexpr (B == 0) MR_STEP8("0", "3");
    if constexpr (B == 1) MR_STEP8("1", "2");
    if constexpr (B == 2) MR_STEP8("2", "1");
    if constexpr (B == 3) MR_STEP8("3", "0");
  } else {
    if constexpr (B == 0) MR_STEP4("0", "3");
    if constexpr (B == 1) MR_STEP4("1", "2");
    if constexpr (B == 2) MR_STEP4("2", "1");
    if constexpr (B == 3) MR_STEP4("3", "0");
  }
#undef MR_STEP8
#undef MR_STEP4
  of = vf, ob = vb;
  vf = pf = nf, vb = pb = nb;
}

// A step of one scan alone (8-connectivity: the other had nothing to do).
template <int B>
__device__ __forceinline__ void column_step1(uint32_t& v, uint32_t& p, uint32_t& o, uint32_t& d, uint32_t m) {
  uint32_t n, t;
#define MR_STEP(BF)                                                                                              \
  asm(MR_DIFF("%2", "%3", "%6") "s_nop 0\n\t" MR_SHR("%0", "%3", "%4") MR_SHL("%1", "%3", "%3") MR_MAX("%0", "%0", "%1") \
          MR_MIN("%0", "%0", "%5", BF)                                                                           \
      : "=&v"(n), "=&v"(t), "+v"(d)                                                                              \
      : "v"(p), "v"(v), "v"(m), "v"(o))
  if constexpr (B == 0) MR_STEP("0");
  if constexpr (B == 1) MR_STEP("1");
  if constexpr (B == 2) MR_STEP("2");
  if constexpr (B == 3) MR_STEP("3");
#undef MR_STEP
  o = v;
  v = p = n;
}
#undef MR_MIN
#undef MR_DIFF
#undef MR_SHR
#undef MR_SHL
#undef MR_MAX

// Steps K .. 15 of chunk C of the forward scan (kF) and of the mirrored chunk of
// the backward scan (kB), on the column v in registers.  pf, pb: the rows before
// this one; of, ob: their old values.
template <int CONN, int C, int K, bool kF, bool kB>
__device__ __forceinline__ void column_steps(uint32_t (&v)[T], uint32_t& df, uint32_t& db, const uint32_t (&ic)[T / 4],
                                             uint32_t pf, uint32_t pb, uint32_t of, uint32_t ob) {
  if constexpr (K < kChunk) {
    constexpr int sf = C * kChunk + K, sb = T - 1 - sf;  // this step's rows
    static_assert((sf & 3) + (sb & 3) == 3, "the backward scan's mask byte mirrors the forward scan's");
    if constexpr (kF && kB)
      column_step2<CONN, (sf & 3)>(v[sf], pf, of, df, ic[sf / 4], v[sb], pb, ob, db, ic[sb / 4]);
    else if constexpr (kF)
      column_step1<(sf & 3)>(v[sf], pf, of, df, ic[sf / 4]);
    else
      column_step1<(sb & 3)>(v[sb], pb, ob, db, ic[sb / 4]);
    column_steps<CONN, C, K + 1, kF, kB>(v, df, db, ic, pf, pb, of, ob);
  } else {
    if constexpr (kF) df = or_diff(of, pf, df);
    if constexpr (kB) db = or_diff(ob, pb, db);
  }
}

// The chunk's steps from the row before it on (the halo acts as zeros).
template <int CONN, int C, bool kF, bool kB>
__device__ __forceinline__ void column_pass(uint32_t (&v)[T], uint32_t& df, uint32_t& db, const uint32_t (&ic)[T / 4]) {
  const uint32_t pf = C > 0 ? v[C > 0 ? C * kChunk - 1 : 0] : 0u, pb = C > 0 ? v[C > 0 ? T - C * kChunk : 0] : 0u;
  column_steps<CONN, C, 0, kF, kB>(v, df, db, ic, pf, pb, pf, pb);
}

template <int C>
__device__ __forceinline__ void store_chunk(WaveLds& L, int l, const uint32_t (&v)[T]) {
#pragma unroll
  for (int k = C * kChunk; k < (C + 1) * kChunk; ++k) L.J[lidx(k, l)] = (uint8_t)v[k];
}

template <int C>
__device__ __forceinline__ void load_chunk(const WaveLds& L, int l, uint32_t (&v)[T]) {
#pragma unroll
  for (int k = C * kChunk; k < (C + 1) * kChunk; ++k) v[k] = L.J[lidx(k, l)];
}

// A chunk of one scan, if it needs it (8-connectivity).
template <int C, bool kF>
__device__ __forceinline__ void column_chunk(const WaveLds& L, int l, uint32_t (&v)[T], const uint32_t (&ic)[T / 4],
                                             Dirty& dm, bool& carry, uint64_t& cols, uint32_t& have, uint32_t& chunks) {
  constexpr int kPos = kF ? C : T / kChunk - 1 - C, kPrev = C == 0 ? kPos : kF ? kPos - 1 : kPos + 1;
  if (!carry && ((kF ? dm.r_cf : dm.r_cb) & chunk_preds(kPos * kChunk, kF)) == 0ull) return;
  if (!(have >> kPos & 1u)) load_chunk<kPos>(L, l, v);
  if (C > 0 && !(have >> kPrev & 1u)) {  // the row before the chunk
    constexpr int r = kF ? kPos * kChunk - (C > 0 ? 1 : 0) : kPos * kChunk + kChunk - (C > 0 ? 0 : 1);
    v[r] = L.J[lidx(r, l)];
  }
  have |= 1u << kPos;
  uint32_t d = 0;
  column_pass<8, C, kF, !kF>(v, d, d, ic);
  const uint64_t c = ballot(d != 0u);
  carry = c != 0ull;
  if (carry) {
    cols |= c;
    chunks |= 1u << kPos;
    (kF ? dm.r_cb : dm.r_cf) |= 0xFFFFull << (kPos * kChunk);
  }
}

// Both column scans (lane = column); returns the columns that changed.  With
// 8-connectivity one after the other: together they would leave the diagonal
// offers of each other's last two passes for another pair (16384^2: 1618 us,
// one after the other 1537).
template <int CONN, bool kDirty>
__device__ __forceinline__ uint64_t column_pair(WaveLds& L, int l, const uint32_t (&ic)[T / 4], Dirty& dm) {
  uint32_t v[T];
  uint64_t cols = 0ull;
  uint32_t chunks = 0u;
  if constexpr (kDirty) {
    bool carry = false;
    uint32_t have = 0u;
    column_chunk<0, true>(L, l, v, ic, dm, carry, cols, have, chunks);
    column_chunk<1, true>(L, l, v, ic, dm, carry, cols, have, chunks);
    column_chunk<2, true>(L, l, v, ic, dm, carry, cols, have, chunks);
    column_chunk<3, true>(L, l, v, ic, dm, carry, cols, have, chunks);
    dm.r_cf = 0ull;
    carry = false;
    column_chunk<0, false>(L, l, v, ic, dm, carry, cols, have, chunks);
    column_chunk<1, false>(L, l, v, ic, dm, carry, cols, have, chunks);
    column_chunk<2, false>(L, l, v, ic, dm, carry, cols, have, chunks);
    column_chunk<3, false>(L, l, v, ic, dm, carry, cols, have, chunks);
    dm.r_cb = 0ull;
  } else {
    load_chunk<0>(L, l, v);
    load_chunk<3>(L, l, v);
    load_chunk<1>(L, l, v);
    load_chunk<2>(L, l, v);
    uint32_t d[T / kChunk] = {0u, 0u, 0u, 0u};
    column_pass<CONN, 0, true, true>(v, d[0], d[3], ic);
    column_pass<CONN, 1, true, true>(v, d[1], d[2], ic);
    column_pass<CONN, 2, true, true>(v, d[2], d[1], ic);
    column_pass<CONN, 3, true, true>(v, d[3], d[0], ic);
#pragma unroll
    for (int c = 0; c < T / kChunk; ++c) {
      const uint64_t b = ballot(d[c] != 0u);
      cols |= b;
      chunks |= b ? 1u << c : 0u;
    }
  }
  if (chunks & 1u) store_chunk<0>(L, l, v);
  if (chunks & 2u) store_chunk<1>(L, l, v);
  if (chunks & 4u) store_chunk<2>(L, l, v);
  if (chunks & 8u) store_chunk<3>(L, l, v);
  wave_sync();
  return cols;
}

// Sweep the tile in LDS until it is locally stable, or `max_it` iterations.
// One iteration is the four axis scans of Algorithm 5, as two pairs: row-wise
// forward (N^{+,0}) and backward (N^{-,0}), column-wise forward (N^{0,+}) and
// backward (N^{0,-}).  Every step is one elementary update J(p) <- max(J(p),
// J(q in the scan's neighbour set)) ^ I(p), so the tile never leaves [J ^ I,
// rho_I(J)].  Halo pixels are sources only, and `fold_halo` applies all their
// offers before the first scan.
//
// When the sweep stops.  With 8-connectivity the scans track what changed
// (`Dirty`): a scan with nothing to do costs nothing, and the tile is stable
// when no scan has anything left.  `all_dirty`: the tile as loaded is not
// known to be locally stable (a seed-pass tile, a tile the sweep cap stopped,
// a full round); otherwise its last visit left it stable and only the border
// pixels the halo raised start dirty.  With 4-connectivity both pairs leave
// their lines stable, so the tile is when a pair after the first changes
// nothing.  `columns_first` picks the first pair, e.g. the one that carries a
// raised halo side into the tile.  Returns true if the tile is locally stable;
// `changed` tells whether any pixel rose.
template <int CONN>
__device__ bool sweep_tile(WaveLds& L, int max_it, uint32_t& iters, bool& changed, bool all_dirty, bool columns_first = false) {
  constexpr bool kDirty = CONN == 8;
  uint64_t rows, cols;
  fold_halo<CONN>(L, rows, cols);
  changed = (rows | cols) != 0ull;
  Dirty dm;
  if (all_dirty || !kDirty) {
    dm.r_cf = dm.r_cb = dm.c_r = ~0ull;
  } else {
    dm.r_cf = dm.r_cb = rows;
    dm.c_r = cols;
  }
  uint32_t ic[T / 4];
  load_mask_column(L, ic);
  const int l = local_copy(lane());
  for (int n = 0; n < 2 * max_it; ++n) {
    if (kDirty && dm.empty()) return true;
    if ((n & 1) == 0) iters++;
    bool rose = false;
    if (((n & 1) != 0) == columns_first) {
      if (!kDirty || dm.c_r) {
        const uint64_t r = row_pair<kDirty>(L, l, dm.c_r);
        dm.c_r = 0ull;
        dm.r_cf |= r;
        dm.r_cb |= r;
        rose = r != 0ull;
      }
    } else if (!kDirty || (dm.r_cf | dm.r_cb)) {
      const uint64_t c = column_pair<CONN, kDirty>(L, l, ic, dm);
      dm.c_r |= c;
      rose = c != 0ull;
    }
    if (rose) changed = true;
    if (!kDirty && !rose && n > 0) return true;
  }
  return kDirty && dm.empty();
}

// Can the (possibly stale) halo pixel (qy, qx) be raised by interior value v?
// J(q) < min(v, I(q)) is the propagation condition of Algorithm 5; the halo J
// may only be lower than the truth, so "no" is always safe.
__device__ __forceinline__ bool halo_raisable(const WaveLds& L, int qy, int qx, uint32_t v) {
  const uint32_t jq = L.J[lidx(qy, qx)], iq = L.I[lidx(qy, qx)];
  return jq < umin(v, iq);
}

// Neighbouring tiles that a change of this visit can raise, as a bit mask:
// bit 0 top, 1 bottom, 2 left, 3 right, 4 top-left, 5 top-right,
// 6 bottom-left, 7 bottom-right.  `old`: the border values before the visit, a
// byte each for top, bottom, left, right (one register over the sweep).
template <int CONN>
__device__ uint32_t border_marks(const WaveLds& L, uint32_t old) {
  const uint32_t ot = old & 0xffu, ob = old >> 8 & 0xffu, ol = old >> 16 & 0xffu, orr = old >> 24;
  const int l = local_copy(lane());
  const uint32_t nt = L.J[lidx(0, l)], nb = L.J[lidx(T - 1, l)];
  const uint32_t nl = L.J[lidx(l, 0)], nr = L.J[lidx(l, T - 1)];
  bool t = false, b = false, lf = false, rt = false;
#pragma unroll
  for (int d = -1; d <= 1; ++d) {
    if (CONN == 4 && d != 0) continue;
    const int c = l + d;
    if (c < 0 || c >= T) continue;
    t |= nt > ot && halo_raisable(L, -1, c, nt);
    b |= nb > ob && halo_raisable(L, T, c, nb);
    lf |= nl > ol && halo_raisable(L, c, -1, nl);
    rt |= nr > orr && halo_raisable(L, c, T, nr);
  }
  uint32_t m = 0;
  if (ballot(t)) m |= 1u;
  if (ballot(b)) m |= 2u;
  if (ballot(lf)) m |= 4u;
  if (ballot(rt)) m |= 8u;
  if (CONN == 8) {
    const uint32_t c00 = L.J[lidx(0, 0)], c0e = L.J[lidx(0, T - 1)];
    const uint32_t ce0 = L.J[lidx(T - 1, 0)], cee = L.J[lidx(T - 1, T - 1)];
    const uint32_t o00 = readlane(ot, 0), o0e = readlane(ot, T - 1);
    const uint32_t oe0 = readlane(ob, 0), oee = readlane(ob, T - 1);
    if (c00 > o00 && halo_raisable(L, -1, -1, c00)) m |= 16u;
    if (c0e > o0e && halo_raisable(L, -1, T, c0e)) m |= 32u;
    if (ce0 > oe0 && halo_raisable(L, T, -1, ce0)) m |= 64u;
    if (cee > oee && halo_raisable(L, T, T, cee)) m |= 128u;
  }
  return m;
}

// Which sides' halo pixels can raise a border pixel of the tile?  (Algorithm
// 5's propagation condition read from the receiving side: J(p) < J(h) and
// J(p) < I(p), for p on the border and h a halo neighbour of p.)  A tile that
// was locally stable after its last visit can only have become raisable this
// way, because only its halo changed since.  Wave-uniform bit mask.
template <int CONN>
__device__ uint32_t border_raisable(const WaveLds& L) {
  const int l = local_copy(lane());
  bool rt = false, rb = false, rl = false, rr = false;
  // p on row 0 (halo row -1), row T-1 (halo row T), column 0 (halo column -1), column T-1 (halo column T)
  const uint32_t pt = L.J[lidx(0, l)], it = L.I[lidx(0, l)];
  const uint32_t pb = L.J[lidx(T - 1, l)], ib = L.I[lidx(T - 1, l)];
  const uint32_t pl = L.J[lidx(l, 0)], il = L.I[lidx(l, 0)];
  const uint32_t pr = L.J[lidx(l, T - 1)], ir = L.I[lidx(l, T - 1)];
#pragma unroll
  for (int d = -1; d <= 1; ++d) {
    if (CONN == 4 && d != 0) continue;
    const int c = l + d;  // -1 .. 64: halo corners included
    rt |= pt < umin(L.J[lidx(-1, c)], it);
    rb |= pb < umin(L.J[lidx(T, c)], ib);
    rl |= pl < umin(L.J[lidx(c, -1)], il);
    rr |= pr < umin(L.J[lidx(c, T)], ir);
  }
  // bits: 0 top, 1 bottom, 2 left, 3 right
  return (ballot(rt) ? 1u : 0u) | (ballot(rb) ? 2u : 0u) | (ballot(rl) ? 4u : 0u) | (ballot(rr) ? 8u : 0u);
}

// ---- raisable-pixel test (full rounds of the bounded mode) -------------------------
// Dense test of the tile in LDS (region loaded with its halo).  Returns
// (wave-uniform) whether some pixel q of the tile can still be raised by a
// neighbour p, i.e. J(q) < J(p) and J(q) < I(q) -- Algorithm 5's propagation
// condition read from the receiving side -- and adds to `seeds` the number of
// pixels p meeting Algorithm 5's seed condition (some neighbour q with
// J(q) < J(p) and J(q) < I(q)).  Lane = column; rows are walked top to
// bottom keeping rows y-1, y, y+1 in registers.

// g(q) = J(q) if q can still rise (J(q) < I(q)), else 256 (never below J(p)).
__device__ __forceinline__ uint32_t gval(uint32_t j, uint32_t i) { return j < i ? j : 256u; }

template <int CONN>
__device__ bool lds_dirty(const WaveLds& L, uint32_t& seeds) {
  const int l = local_copy(lane());
  const int hc = l == 0 ? -1 : T;  // fill column: lane 0 uses column -1, lane 63 column 64
  uint32_t jp = L.J[lidx(-1, l)], ip = L.I[lidx(-1, l)], fjp = L.J[lidx(-1, hc)], fip = L.I[lidx(-1, hc)];
  uint32_t jc = L.J[lidx(0, l)], ic = L.I[lidx(0, l)], fjc = L.J[lidx(0, hc)], fic = L.I[lidx(0, hc)];
  bool any = false;
  uint32_t cnt = 0;
#pragma unroll
  for (int c = 0; c < T / kChunk; ++c) {
    uint32_t nj[kChunk], ni[kChunk], nfj[kChunk], nfi[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      const int y = c * kChunk + k + 1;
      nj[k] = L.J[lidx(y, l)];
      ni[k] = L.I[lidx(y, l)];
      nfj[k] = L.J[lidx(y, hc)];
      nfi[k] = L.I[lidx(y, hc)];
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      const uint32_t jn = nj[k], in = ni[k], fjn = nfj[k], fin = nfi[k];
      uint32_t m = umax(umax(jp, jn), umax(from_left(jc, fjc), from_right(jc, fjc)));
      const uint32_t gc = gval(jc, ic), gfc = gval(fjc, fic);
      uint32_t g = umin(umin(gval(jp, ip), gval(jn, in)), umin(from_left(gc, gfc), from_right(gc, gfc)));
      if (CONN == 8) {
        m = umax(m, umax(umax(from_left(jp, fjp), from_right(jp, fjp)), umax(from_left(jn, fjn), from_right(jn, fjn))));
        const uint32_t gp = gval(jp, ip), gfp = gval(fjp, fip), gn = gval(jn, in), gfn = gval(fjn, fin);
        g = umin(g, umin(umin(from_left(gp, gfp), from_right(gp, gfp)), umin(from_left(gn, gfn), from_right(gn, gfn))));
      }
      any |= jc < umin(m, ic);
      cnt += (uint32_t)__popcll(ballot(jc > g));
      jp = jc; ip = ic; fjp = fjc; fip = fic;
      jc = jn; ic = in; fjc = fjn; fic = fin;
    }
    asm volatile("" ::: "memory");
  }
  seeds += cnt;
  return ballot(any) != 0;
}

// ---- persistent propagation -----------------------------------------------------------
// The frontier of round r+1 while round r runs: the parity's flags and list,
// the sub-list this workgroup appends to, its capacity and lost flag.
struct Next {
  uint32_t* flags;
  uint32_t* list;
  uint32_t* count;
  uint32_t cap;
  uint32_t* lost;
};

__device__ __forceinline__ Next next_frontier(const MrArgs& a, uint32_t r) {
  const bool bounded = a.list_cap < a.ntiles;
  const uint32_t par = (r + 1u) & 1u, shard = bounded ? 0u : (blockIdx.x & (uint32_t)(kShards - 1));
  Next n;
  n.flags = a.flags + (size_t)par * a.ntiles;
  n.list = a.lists + ((size_t)par * kShards + shard) * a.ntiles;
  n.count = shard_count(a.counts, (r + 1u) % 3u, shard);
  n.cap = bounded ? a.list_cap : a.ntiles;
  n.lost = a.lost + par * 64u;
  return n;
}

// Flag the neighbours named by border mask m (see border_marks) and, if
// `unsettled`, the tile itself, for the next round (lanes 0..8 of the wave).
__device__ __forceinline__ void mark_reach(WaveStage& s, const Next& nx, const TileRef& tr, uint32_t m, bool unsettled,
                                           uint32_t* appended) {
  const int l = local_copy(lane());
  int dy = 0, dx = 0;
  bool want = false;
  if (l < 8) {
    // bit order of border_marks: top, bottom, left, right, tl, tr, bl, br
    want = (m >> l) & 1u;
    dy = l < 2 ? (l == 0 ? -1 : 1) : (l < 4 ? 0 : (l < 6 ? -1 : 1));
    dx = l < 2 ? 0 : (l < 4 ? (l == 2 ? -1 : 1) : ((l & 1) ? 1 : -1));
  } else if (l == 8) {
    want = unsettled;
  }
  const int ny = tr.ty + dy, nx_ = tr.tx + dx;
  want = want && ny >= 0 && ny < tr.j.tiles_y && nx_ >= 0 && nx_ < tr.j.tiles_x;
  shard_mark(s, want, tr.j.tile_base + (uint32_t)(ny * tr.j.tiles_x + nx_), nx.flags, nx.list, nx.count, nx.cap, nx.lost,
             appended);
}

// A wave's counters over the kernel.
struct Counters {
  uint32_t visits = 0, iters = 0, seeds = 0;
};

enum class Visit { kSeed, kListed, kCheck };

// One visit of a tile: load it with its halo, sweep to local stability, write
// back, and flag the neighbouring tiles a border change can raise (and the
// tile itself if the sweep cap stopped it).
//
// kSeed (round 0): the tile comes from the clamped marker.  In strip order
// (`fresh_top`: the tile above was written by this wave just before) the halo
// row above comes from the output; `below_next`: the tile below is this wave's
// next tile and will read this one's result, so it need not be flagged for this
// tile's bottom edge.
//
// kListed: a tile that its last visit left stable needs work only if its new
// halo can raise its border (`border_raisable`); kCheck (full rounds): the
// whole tile is tested instead.
//
// One function for the three, called from one place: the sweep is some 40 KB of
// code, and a copy for each would not fit the instruction cache together.
template <int CONN>
__device__ __forceinline__ void visit_tile(WaveLds& L, WaveStage& s, uint32_t round, uint32_t t,
                                           Visit how, bool fresh_top, bool below_next, bool few, uint32_t* appended,
                                           Counters& n) {
  const MrArgs a = kernel_args<MrArgs>();
  const TileRef tr = tile_ref(a, t);
  bool columns_first = false, all_dirty = true;
  if (how == Visit::kSeed) {
    if (fresh_top) drain();  // this wave's stores of the tile above are complete
    load_region<true>(tr, L, fresh_top);
  } else {
    const uint32_t uns = how == Visit::kListed && lane() == 0 ? cload(a.unsettled + t) : 0u;
    if (CONN == 8 && how == Visit::kListed && !few) {
      // About a third of the listed 8-connected tiles turn out to need no
      // work: load the frame first and the interior only if needed.  Nearly
      // every listed 4-connected tile needs work, and the second round trip
      // measured slower there (1.85 against 1.81 ms): one load.  With few tiles
      // in the round (at most one a workgroup) the round trip counts, not the bytes.
      load_frame(tr, L, a.cols, a.ntiles * 256u, t);
    } else {
      load_region<false>(tr, L, false, a.cols, a.ntiles * 256u, t);
    }
    if (how == Visit::kCheck) {
      if (!lds_dirty<CONN>(L, n.seeds)) return;
    } else {
      const uint32_t sides = border_raisable<CONN>(L);
      all_dirty = readlane(uns, 0) != 0u;
      if (!all_dirty && sides == 0u) return;
      if (CONN == 8 && !few) load_interior(tr, L);
      columns_first = (sides & 3u) != 0u;  // the scans that lead away from a raisable top or bottom
    }
  }
  const int l = local_copy(lane());
  const uint32_t old = L.J[lidx(0, l)] | (uint32_t)L.J[lidx(T - 1, l)] << 8 | (uint32_t)L.J[lidx(l, 0)] << 16 |
                       (uint32_t)L.J[lidx(l, T - 1)] << 24;
  const bool seed = how == Visit::kSeed;
  bool changed;
  const bool stable =
      sweep_tile<CONN>(L, seed ? a.seed_sweeps : a.max_sweeps, n.iters, changed, all_dirty, columns_first);
  if (!seed) n.visits++;
  const Next nx = next_frontier(a, round);
  if (lane() == 0) cstore(a.unsettled + t, stable ? 0u : 1u);
  if (changed || seed) {
    store_tile(tr, L);
    store_cols(a, t, L, seed);
  }
  uint32_t m = changed ? border_marks<CONN>(L, old) : 0u;
  if (below_next) m &= ~2u;  // bit 1: bottom
  mark_reach(s, nx, tr, m, !stable, appended);
}

// Tiles per strip of the seed pass.  A strip carries the flood down a column of
// tiles, but a strip for every wave has no slack, where of single tiles in row order
// a workgroup's faster waves take more.  With 8-connectivity strips are taken where
// they come out even, at least 95% of the waves' steps being tiles, as was measured
// with four waves a workgroup (us, strips and single: 16384^2 1413, 1480; 12000^2
// 922, 965; 32768^2 4888, 5039).  With eight, the default, they still gain up to 2%
// where every wave has a whole strip (16384^2 1379, 1408; 12000^2 658, 680), but at
// most other sizes single tiles are better, by up to 14% and the more the longer the
// strips (20000 x 17000 1645, 1484; 32768^2 3721, 3487; 15189 x 16844 1710, 1593;
// 8633 x 16884 1021, 1018): a line of its own for eight waves is open.  Where they
// come out uneven (24000^2 2187, 2043; 65536 x 65600, where 4100 strips meet 4096
// waves, 14360, 12887), and with 4-connectivity (16384^2 1188, 1158; 24000^2 2600,
// 2409; 20000 x 17000 2020, 1837; 12000^2 794, 785), single tiles.
__device__ __forceinline__ uint32_t auto_strip(const MrArgs& a, int conn, uint32_t nw) {
  const uint32_t S = (a.ntiles + nw - 1u) / nw;
  const uint32_t tx_n = (uint32_t)a.job0.tiles_x, ty_n = (uint32_t)a.job0.tiles_y;
  const uint32_t nstrips = tx_n * ((ty_n + S - 1u) / S), passes = (nstrips + nw - 1u) / nw;
  return conn == 8 && (uint64_t)a.ntiles * 20u >= (uint64_t)nw * S * passes * 19u ? S : 1u;
}

// Round 0 is the seed pass over every tile; round r >= 1 visits the tiles
// listed in round r-1 and lists the tiles of round r+1 (parity (r+1)&1,
// count slot (r+1)%3).  The list is split over kShards sub-lists, one per
// group of workgroups; a group's sub-list is cut into one share per
// workgroup (WgShare).  Bounded mode (a capacity below
// the tile count) uses one sub-list of that capacity; a round whose list
// lost tiles is replaced by a full round that visits every tile holding a
// raisable pixel (all flags cleared first), restarting from the current
// image.  The flags and the counts must be zero when the kernel starts.
// WPB waves per workgroup.
template <int CONN, int WPB>
__global__ __launch_bounds__(64 * WPB, 4) void k_propagate(MrArgs a) {
  __shared__ WaveLds lds[WPB];
  __shared__ uint32_t stage_mem[WPB][kStageCap];
  __shared__ uint32_t cnt[kShards];
  __shared__ uint32_t lost_sh, next_sh, appended_sh;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  WaveLds& L = lds[w];
  const uint32_t depth = a.stage_depth > 0u && a.stage_depth < (uint32_t)kStageCap ? a.stage_depth : (uint32_t)kStageCap;
  WaveStage s = {stage_mem[w], depth, 0u};
  L.J[lidx(lane() - 1, kZeroCol)] = 0;  // rows -1..62
  if (lane() < 2) L.J[lidx(T - 1 + lane(), kZeroCol)] = 0;  // rows 63, 64
  if (threadIdx.x == 0) next_sh = appended_sh = 0u;
  Appended app = {&appended_sh, cnt, &next_sh, 0u};
  const bool bounded = a.list_cap < a.ntiles;
  __syncthreads();
  const uint32_t nw = gridDim.x * WPB;  // waves of the grid
  const uint32_t cap = a.list_cap < a.ntiles ? a.list_cap : a.ntiles;
  uint32_t gen = 0, nclk = 0;
  uint32_t rounds = 0, restarts = 0, first = 0;
  Counters n_;
  clock_stamp(a.clock, nclk);
  // Seed pass, strip order (one image): each wave seeds vertical strips of S
  // tiles top to bottom, so the flood crosses the horizontal tile edges inside
  // the seed pass.  The strips are shared by the waves of each workgroup.
  const bool strips = a.njobs == 1u;
  const uint32_t S = !strips ? 1u : a.seed_strip > 0u ? a.seed_strip : auto_strip(a, CONN, nw);
  for (uint32_t r = 0;; ++r) {
    const uint32_t par = r & 1u;
    bool full = false;
    uint32_t n = a.ntiles;
    if (r > 0u) {
      // The barrier left in cnt what each group appended.  Only a bounded list
      // can have lost some.
      n = 0;
      for (int x = 0; x < kShards; ++x) n += cnt[x];
      if (bounded) {
        if (n > cap) n = cap;
        if (threadIdx.x == 0) lost_sh = cload(a.lost + par * 64u);
        __syncthreads();
        full = lost_sh != 0u;
      }
      if (!full && n == 0u) break;
    }
    round_work(a.clock, r, full ? a.ntiles : n);
    if (r >= kMaxRounds) {  // safety limit: report instead of spinning on a logic error
      if (blockIdx.x == 0 && threadIdx.x == 0) stat_add(a.stats, kStatError, 1ull);
      break;
    }
    if (full) {
      if (!grid_barrier(a.bar, gen, a.stats)) break;  // everyone has read the decision
      for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < 2u * a.ntiles; i += gridDim.x * blockDim.x)
        cstore(a.flags + i, 0u);
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        cstore(a.lost, 0u);
        cstore(a.lost + 64, 0u);
        restarts++;
      }
      if (!grid_barrier(a.bar, gen, a.stats)) break;
    }
    // The counts of round r+2 are reused: clear them now (they were last read
    // in round r-1, and are next appended to in round r+1, after this round's barrier).
    if (r > 0u && blockIdx.x == 0 && threadIdx.x < (unsigned)kShards)
      cstore(shard_count(a.counts, (r + 2u) % 3u, threadIdx.x), 0u);
    const uint32_t before = n_.visits;
    const uint32_t* lists = a.lists + (size_t)par * kShards * a.ntiles;
    uint32_t* flg = a.flags + (size_t)par * a.ntiles;
    const uint32_t tx_n = (uint32_t)a.job0.tiles_x, ty_n = (uint32_t)a.job0.tiles_y;  // strips only
    // Items: strips or tiles (seed pass, full round), entries of the lists.
    // XCD x visits the tiles XCD x listed (a bounded list is one sub-list:
    // then the whole list is cut over the grid).  With at most one item per
    // workgroup the first wave of workgroup b of the XCD takes item b: no
    // counter in LDS, and tiles on different CUs.
    const uint32_t items = r == 0u && strips ? tx_n * ((ty_n + S - 1u) / S) : full ? a.ntiles : n;
    const bool own = r > 0u && !full && !bounded && gridDim.x >= kXcds;
    const uint32_t grp = own ? blockIdx.x % kXcds : 0u, rank = blockIdx.x / kXcds;
    const uint32_t mine = own ? cnt[grp] : 0u;
    const bool few = own && n <= gridDim.x && mine <= xcd_groups(grp);
    const WgShare share = own ? share_of(0u, mine, &next_sh) : wg_share(items, &next_sh);
    const Visit how = r == 0u ? Visit::kSeed : full ? Visit::kCheck : Visit::kListed;
    uint32_t t = 0, left = 0;  // seed pass: the tile, and how many of its strip follow
    bool fresh = false, taken = false;
    for (;;) {
      if (left > 0u) {
        --left;
        t += tx_n;
      } else {
        uint32_t i = rank;
        if (few) {
          if (w != 0 || rank >= mine || taken) break;
          taken = true;
        } else if (!share.take(i)) {
          break;
        }
        t = i;
        if (how == Visit::kListed) {
          t = own || bounded ? cload(lists + (size_t)grp * a.ntiles + i) : shard_item(lists, a.ntiles, cnt, i);
          t = readlane(t, 0);
          if (lane() == 0) cstore(flg + t, 0u);
        } else if (how == Visit::kSeed && strips) {
          const uint32_t ty0 = i / tx_n * S;
          t = ty0 * tx_n + i % tx_n;
          left = (ty0 + S < ty_n ? ty0 + S : ty_n) - ty0 - 1u;
        }
        fresh = false;
      }
      // Right-edge tiles of widths not a multiple of 16 read bytes: stale halo there.
      const bool below = left > 0u && !(a.job0.w % 16 != 0 && t % tx_n + 1u == tx_n);
      visit_tile<CONN>(L, s, r, t, how, fresh, below, few, &appended_sh, n_);
      fresh = below;
    }
    {
      const MrArgs b = kernel_args<MrArgs>();
      const Next nx = next_frontier(b, r);
      shard_flush(s, nx.list, nx.count, nx.cap, nx.flags, nx.lost, &appended_sh);
    }
    if (r == 1u) first = n_.visits - before;
    if (r > 0u) rounds++;
    const bool ok = grid_barrier(a.bar, gen, a.stats, &app);
    clock_stamp(a.clock, nclk);
    if (!ok || a.seed_only != 0u) break;
  }
  if (lane() == 0) {
    stat_add(a.stats, kStatSeeds, (unsigned long long)first);
    stat_add(a.stats, kStatItems, n_.visits);
    stat_add(a.stats, kStatSweeps, n_.iters);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    stat_add(a.stats, kStatRounds, rounds);
    stat_add(a.stats, kStatRestarts, restarts);
  }
}

// Image of every global tile, by binary search over the images' first tiles.
__global__ void k_tile_job(const MrJob* jobs, uint32_t njobs, uint32_t* tile_job, uint32_t ntiles) {
  for (uint32_t t = blockIdx.x * blockDim.x + threadIdx.x; t < ntiles; t += gridDim.x * blockDim.x) {
    uint32_t lo = 0, hi = njobs;  // last job with tile_base <= t
    while (hi - lo > 1u) {
      const uint32_t mid = (lo + hi) >> 1;
      if (jobs[mid].tile_base <= t) lo = mid; else hi = mid;
    }
    tile_job[t] = lo;
  }
}

}  // namespace mr

// ---- host-side launch -----------------------------------------------------------------
int mr_launch(const MrArgs& a, int conn, int persistent_blocks, hipStream_t stream, Recorder* rec, const char** err) {
  using namespace mr;
  if (a.njobs > 1u) {
    const uint32_t b = (a.ntiles + 255u) / 256u;
    hipLaunchKernelGGL(k_tile_job, dim3(b < 1024u ? b : 1024u), dim3(256), 0, stream, a.jobs, a.njobs, a.tile_job, a.ntiles);
    if (hipGetLastError() != hipSuccess) {
      *err = "tile map launch failed";
      return -1;
    }
  }
  const int wpb = a.wg_waves == 8u ? 8 : 4;
  void* fn = wpb == 8 ? (conn == 8 ? reinterpret_cast<void*>(&k_propagate<8, 8>) : reinterpret_cast<void*>(&k_propagate<4, 8>))
                      : (conn == 8 ? reinterpret_cast<void*>(&k_propagate<8, 4>) : reinterpret_cast<void*>(&k_propagate<4, 4>));
  int dev = 0, per_cu = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 64 * wpb, 0) != hipSuccess || per_cu < 1) {
    *err = "occupancy query failed";
    return -1;
  }
  uint32_t blocks = persistent_grid(fn, per_cu, cus, 16 / wpb);
  if (persistent_blocks > 0 && (uint32_t)persistent_blocks < blocks) blocks = (uint32_t)persistent_blocks;
  MrArgs args = a;
  void* kargs[] = {&args};
  rec->begin(3, stream);
  const hipError_t le = launch_persistent(fn, blocks, kargs, stream, 64 * wpb);
  rec->end(stream);
  if (le != hipSuccess) {
    *err = "propagation launch failed";
    return -1;
  }
  return 0;
}

}  // namespace iwpp
