// Exact Euclidean distance transform (iwpp_edt_exact).
//
// The propagation EDT of Sec. 2.2 is an approximation; the paper notes that
// exact distances need extra work beyond the 8-neighbour propagation.  This
// is the exact transform, separable as in Meijster, Roerdink and Hesselink
// (2000): with r(x') the row of column x's nearest feature as seen from row y,
// the squared distance at (y, x) is the minimum over the columns x' of
//     F(x, x') = (x - x')^2 + (y - r(x'))^2.
//   1. columns: 64-row segments of a column as bit masks (k_mask), from which
//      every pixel's nearest feature in its own column follows by counting
//      leading and trailing zeros (k_col);
//   2. rows: the minimising column, ties to the smaller one, never decreases
//      with x (F(x, a) - F(x, b) is monotone in x).  So once it is known at
//      the multiples of 2s it is searched for at the odd multiples of s only
//      between its two neighbours' columns, for s halving down to 1 (k_row).
// All arithmetic is integer; the squared distance is exact and the nearest
// feature is one at exactly that distance (ties: the smaller column, then the
// upper row).
//
// Bound: 13 bytes a pixel move (mask 1, column rows 2 + 2, outputs 8, and the
// segment masks), 43 us for 4096^2 at the copy rate.  Measured there (30%
// features): k_mask 7 us, k_col 17 us, k_row 250 us, bound by the searches'
// LDS round trips and integer arithmetic (one lane per row with a stack of
// parabolas in memory, which this replaces: 5.65 ms for the whole call).
#include <hip/hip_runtime.h>

#include <string>

#include "../../include/iwpp.h"
#include "iwpp_device.hpp"
#include "iwpp_internal.hpp"
#include "iwpp_runtime.hpp"

namespace iwpp {
namespace xedt {

constexpr int kSeg = 64;      // rows per column segment: one mask bit each
constexpr int kSuper = 16;    // segments per super-segment, and waves of a k_mask workgroup
constexpr uint32_t kNone = 0xFFFFu;  // no feature (rows are below 46340)
constexpr int kStride = 16;   // first anchors of a row: multiples of this
constexpr int kReach = 64;    // columns an anchor's outward search may go before the row takes the general path
constexpr int kShort = 8;     // ranges that every lane searches for itself
constexpr int kFew = 16;      // longer ranges that the wave shares one after another rather than wait for them
constexpr int kSerial = 64;   // longest range one lane searches alone
constexpr uint32_t kFar = 46341u;  // stands for "no feature in the column": its square is above every real one,
                                   // and stays below 2^32 with a column distance's square added

// LDS of the row pass for rows w wide: 3 bytes a column.
constexpr uint32_t row_lds(uint32_t w) { return 2u * (w + (w + 1u) / 2u); }
constexpr uint32_t kMaxRowLds = row_lds(46340);  // the widest row accepted
static_assert(kMaxRowLds <= 160u * 1024u, "a CU's LDS");

struct XArgs {
  const uint8_t* bin;  // 0 = feature
  int32_t* sqdist;
  int32_t* nearest;
  unsigned long long* mask;  // [nseg][w] feature rows of the segment, bit = row
  uint16_t* some;            // [nsuper][w] the super-segment's segments that hold a feature
  uint16_t* frow;            // [h][w] row of the nearest feature in the pixel's column, or kNone
  int32_t h, w, nseg;
};

// Segment masks: lane = column, one segment per wave, a super-segment per
// workgroup, so that the super-segment's summary is gathered in LDS (a
// device-scope atomic per segment would cost more than the pass itself).
__global__ __launch_bounds__(64 * kSuper) void k_mask(XArgs a) {
  __shared__ uint32_t some[64];
  const int l = lane(), k = (int)threadIdx.x / 64;
  const int x = blockIdx.x * 64 + l, s = blockIdx.y * kSuper + k;
  if (threadIdx.x < 64) some[l] = 0u;
  __syncthreads();
  if (x < a.w && s < a.nseg) {
    const uint8_t* p = a.bin + (size_t)s * kSeg * (uint32_t)a.w + (uint32_t)x;
    const int n = a.h - s * kSeg < kSeg ? a.h - s * kSeg : kSeg;
    unsigned long long m = 0;
    if (n == kSeg) {
#pragma unroll 16
      for (int r = 0; r < kSeg; ++r) m |= (unsigned long long)(p[(size_t)r * (uint32_t)a.w] == 0) << r;
    } else {
      for (int r = 0; r < n; ++r) m |= (unsigned long long)(p[(size_t)r * (uint32_t)a.w] == 0) << r;
    }
    a.mask[(size_t)s * (uint32_t)a.w + (uint32_t)x] = m;
    if (m) atomicOr(&some[l], 1u << k);
  }
  __syncthreads();
  if (threadIdx.x < 64 && x < a.w) a.some[(size_t)blockIdx.y * (uint32_t)a.w + (uint32_t)x] = (uint16_t)some[l];
}

// The nearest feature row in its column for every pixel of a segment (lane =
// column): the last feature at or above, the first at or below; the closer
// wins, the upper on a tie.  The nearest segments above and below that hold a
// feature come from the super-segment summaries.
__global__ __launch_bounds__(256) void k_col(XArgs a) {
  const int x = blockIdx.x * 256 + (int)threadIdx.x, s = blockIdx.y;
  if (x >= a.w) return;
  const size_t w = (size_t)(uint32_t)a.w;
  const unsigned long long m = a.mask[(size_t)s * w + (uint32_t)x];
  const int nsuper = (a.nseg + kSuper - 1) / kSuper, k = s % kSuper;
  int above = -1, below = -1;  // feature rows outside the segment
  {
    int t = s / kSuper;
    uint32_t b = a.some[(size_t)t * w + (uint32_t)x] & ((1u << k) - 1u);
    while (b == 0u && --t >= 0) b = a.some[(size_t)t * w + (uint32_t)x];
    if (b != 0u) {
      const int u = t * kSuper + 31 - __clz((int)b);
      above = u * kSeg + 63 - __clzll((long long)a.mask[(size_t)u * w + (uint32_t)x]);
    }
  }
  {
    int t = s / kSuper;
    uint32_t b = a.some[(size_t)t * w + (uint32_t)x] & ~((2u << k) - 1u);
    while (b == 0u && ++t < nsuper) b = a.some[(size_t)t * w + (uint32_t)x];
    if (b != 0u) {
      const int u = t * kSuper + __ffs((int)b) - 1;
      below = u * kSeg + __ffsll((long long)a.mask[(size_t)u * w + (uint32_t)x]) - 1;
    }
  }
  const int y0 = s * kSeg, n = a.h - y0 < kSeg ? a.h - y0 : kSeg;
  uint16_t* out = a.frow + (size_t)y0 * w + (uint32_t)x;
  for (int r = 0; r < n; ++r) {
    const int y = y0 + r;
    if ((m >> r) & 1ull) above = y;
    const unsigned long long rest = m >> r;
    const int dn = rest ? y + __ffsll((long long)rest) - 1 : below;
    const int f = above < 0 ? dn : (dn < 0 || y - above <= dn - y ? above : dn);
    out[(size_t)r * w] = f < 0 ? (uint16_t)kNone : (uint16_t)f;
  }
}

// F(x, c) from the columns' row distances (kFar for a column without
// features: then 2^31 or more, which no real value reaches).
__device__ __forceinline__ uint32_t dist(const uint16_t* g, int x, int c) {
  const int dx = x - c;
  return (uint32_t)__mul24(dx, dx) + (uint32_t)__umul24(g[c], g[c]);
}

// Columns farther from x than the square root of a distance some column
// reaches cannot hold the minimum.
__device__ __forceinline__ int reach(uint32_t d) { return (int)__fsqrt_rn((float)d) + 1; }

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  auto step = [&](uint32_t o) { v = v < o ? v : o; };
  step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x111 /* row_shr:1 */, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x112 /* row_shr:2 */, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x114 /* row_shr:4 */, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x118 /* row_shr:8 */, 0xf, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142 /* row_bcast:15 */, 0xa, 0xf, false));
  step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143 /* row_bcast:31 */, 0xc, 0xf, false));
  return readlane(v, kWave - 1);
}

// Pass 2: one workgroup per row, the columns' row distances and the minimising
// columns of its even pixels in LDS (3 bytes a column: 139 KB of the CU's 160
// for the widest rows).
//
// First the anchors (multiples of kStride), each by a search outward from x
// that ends once no column farther out can win; where one would go past
// kReach (sparse images) the row takes the general path instead: the halving
// starts from the whole row, so that every level reads each column about once
// however far the features lie.
//
// Most ranges are a few columns (the nearest feature moves slowly along a
// shape), a few per wave span the gap between two shapes.  The wave searches
// those few together, a lane per column, instead of waiting for one lane (up
// to 64 lanes waiting for the longest range: 407 us against 250).
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_row(XArgs a) {
  extern __shared__ uint16_t lds[];
  uint16_t* g = lds;          // [w]
  uint16_t* arg = lds + a.w;  // [(w + 1) / 2]: even pixels
  const int y = blockIdx.x, W = a.w;
  const uint16_t* src = a.frow + (size_t)y * (uint32_t)W;
  for (int x = threadIdx.x; x < W; x += kThreads) {
    const uint32_t r = src[x];
    g[x] = (uint16_t)(r == kNone ? kFar : (uint32_t)(y > (int)r ? y - (int)r : (int)r - y));
  }
  __syncthreads();

  // The minimising column in [lo, hi]: called by whole waves.
  auto search = [&](bool on, int x, int lo, int hi) -> int {
    if (on && hi - lo > kShort) {
      const uint32_t d0 = dist(g, x, lo), d1 = dist(g, x, hi), d2 = dist(g, x, x);
      const uint32_t d = d0 < d1 ? (d0 < d2 ? d0 : d2) : (d1 < d2 ? d1 : d2);
      if (d < 0x80000000u) {
        const int m = reach(d);
        lo = lo > x - m ? lo : x - m;
        hi = hi < x + m ? hi : x + m;
      }
    }
    int best = lo;
    const uint64_t few = ballot(on && hi - lo > kShort);
    const bool shared = on && hi - lo > (__popcll(few) <= kFew ? kShort : kSerial);
    if (on && !shared) {
      uint32_t bd = dist(g, x, lo);
      for (int c = lo + 1; c <= hi; ++c) {
        const uint32_t d = dist(g, x, c);
        if (d < bd) {
          bd = d;
          best = c;
        }
      }
    }
    for (uint64_t todo = ballot(shared); todo; todo &= todo - 1) {
      const int who = (int)__builtin_ctzll(todo);
      const int sx = (int)readlane((uint32_t)x, who), sl = (int)readlane((uint32_t)lo, who), sh = (int)readlane((uint32_t)hi, who);
      uint32_t bd = 0xFFFFFFFFu;
      uint32_t bc = 0xFFFFFFFFu;
#pragma unroll 4
      for (int c = sl + lane(); c <= sh; c += kWave) {
        const uint32_t d = dist(g, sx, c);
        if (d < bd) {
          bd = d;
          bc = (uint32_t)c;
        }
      }
      const uint32_t m = wave_min(bd);
      const int at = sh - sl < kWave ? sl + (int)__builtin_ctzll(ballot(bd == m))
                                     : (int)wave_min(bd == m ? bc : 0xFFFFFFFFu);
      if (lane() == who) best = at;
    }
    return best;
  };

  const int w0 = (int)(threadIdx.x & ~63u);  // the wave's first thread
  bool far = false;
  for (int x = (int)threadIdx.x * kStride; x < W; x += kThreads * kStride) {
    uint32_t bd = dist(g, x, x);
    int best = x;
    for (int dx = 1; (uint32_t)(dx * dx) <= bd; ++dx) {
      const bool l = x - dx >= 0, r = x + dx < W;
      if (!l && !r) break;
      if (dx > kReach) {
        far = true;
        break;
      }
      const uint32_t dl = l ? dist(g, x, x - dx) : 0xFFFFFFFFu, dr = r ? dist(g, x, x + dx) : 0xFFFFFFFFu;
      if (dl <= bd) {  // a smaller column than any seen so far: it takes ties
        bd = dl;
        best = x - dx;
      }
      if (dr < bd) {
        bd = dr;
        best = x + dx;
      }
    }
    arg[x >> 1] = (uint16_t)best;
  }
  int s = kStride / 2;
  if (__syncthreads_or(far)) {
    if (w0 == 0) {
      const int best = search(lane() == 0, 0, 0, W - 1);
      if (lane() == 0) arg[0] = (uint16_t)best;
    }
    s = 2;
    while (2 * s < W) s *= 2;
    __syncthreads();
  }
  for (; s > 1; s >>= 1) {
    const int n = W > s ? (W - 1 - s) / (2 * s) + 1 : 0;  // odd multiples of s below W
    for (int i0 = 0; i0 < n; i0 += kThreads) {
      // dealt to the waves in turn: the few anchors of the first levels have long ranges
      const int i = i0 + lane() * (kThreads / kWave) + w0 / kWave, x = s * (2 * i + 1);
      const bool on = i < n;
      const int lo = on ? arg[(x - s) >> 1] : 0, hi = on && x + s < W ? arg[(x + s) >> 1] : W - 1;
      const int best = search(on, x, lo, hi);
      if (on) arg[x >> 1] = (uint16_t)best;
    }
    __syncthreads();
  }
  // Odd pixels, and the output of both.
  int32_t* sq = a.sqdist + (size_t)y * (uint32_t)W;
  int32_t* nr = a.nearest + (size_t)y * (uint32_t)W;
  for (int i0 = w0; 2 * i0 < W; i0 += kThreads) {
    const int i = i0 + lane(), x = 2 * i;
    const bool on = x + 1 < W;
    const int c0 = x < W ? arg[i] : 0, hi = x + 2 < W ? arg[i + 1] : W - 1;
    const int c1 = search(on, x + 1, c0, hi);
    auto put = [&](int px, int c) {
      const uint32_t r = src[c], d = dist(g, px, c);
      sq[px] = r == kNone ? -1 : (int32_t)d;
      nr[px] = r == kNone ? -1 : (int32_t)r * W + c;
    };
    if (x < W) put(x, c0);
    if (on) put(x + 1, c1);
  }
}

}  // namespace xedt
}  // namespace iwpp

using namespace iwpp::rt;

extern "C" int32_t iwpp_edt_exact(iwpp_ctx* ctx, const uint8_t* binary, int32_t* sqdist, int32_t* nearest,
                                  int32_t height, int32_t width, void* stream) {
  using namespace iwpp;
  if (!ctx) return IWPP_EINVAL;
  if (ctx->server) return fail(ctx, IWPP_EBUSY, "edt_exact: the context is serving");
  if (!binary || !sqdist || !nearest) return fail(ctx, IWPP_EINVAL, "edt_exact: NULL image pointer");
  // the same argument rules as iwpp_edt (conn is irrelevant here)
  iwpp_job j{IWPP_OP_EDT, 8, height, width, binary, nullptr, sqdist, nearest};
  Plan plan;
  int32_t rc = build_plan(ctx, &j, 1, "edt_exact", plan);
  if (rc != IWPP_OK) return rc;
  const size_t np = (size_t)height * (size_t)width;
  const int nseg = (height + xedt::kSeg - 1) / xedt::kSeg, nsuper = (nseg + xedt::kSuper - 1) / xedt::kSuper;
  const size_t fb = align256(2 * np), mb = align256(8 * (size_t)nseg * (size_t)width);
  DeviceGuard g(ctx->device);
  if (!g.ok) return fail(ctx, IWPP_EDEVICE, "edt_exact: cannot select the context's device");
  if ((rc = ensure_scratch(ctx, fb + mb + align256(2 * (size_t)nsuper * (size_t)width))) != IWPP_OK) return rc;
  xedt::XArgs a{};
  a.bin = binary;
  a.sqdist = sqdist;
  a.nearest = nearest;
  a.mask = reinterpret_cast<unsigned long long*>(ctx->scratch);
  a.frow = reinterpret_cast<uint16_t*>(ctx->scratch + mb);
  a.some = reinterpret_cast<uint16_t*>(ctx->scratch + mb + fb);
  a.h = height;
  a.w = width;
  a.nseg = nseg;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // Rows wider than 8192 take 1024 threads: their 3 bytes of LDS a column leave
  // room for few workgroups per CU.  Rows up to 512 take one wave each.
  const int threads = width > 8192 ? 1024 : (width > 512 ? 256 : 64);
  const uint32_t lds = xedt::row_lds((uint32_t)width);
  void (*row)(xedt::XArgs) = threads == 1024 ? &xedt::k_row<1024> : (threads == 256 ? &xedt::k_row<256> : &xedt::k_row<64>);
  // The kernel's limit belongs to the process: always the same value, so that a call
  // of another thread with narrower rows cannot lower it between here and the launch.
  if (lds > 64u * 1024u && hipFuncSetAttribute(reinterpret_cast<const void*>(row), hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)xedt::kMaxRowLds) != hipSuccess) {
    (void)hipGetLastError();
    return fail(ctx, IWPP_EDEVICE, "edt_exact: the row pass's LDS is not available");
  }
  ctx->rec.begin(IWPP_K_XEDT, st);
  hipLaunchKernelGGL(xedt::k_mask, dim3((unsigned)((width + 63) / 64), (unsigned)nsuper), dim3(64 * xedt::kSuper), 0, st, a);
  hipLaunchKernelGGL(xedt::k_col, dim3((unsigned)((width + 255) / 256), (unsigned)nseg), dim3(256), 0, st, a);
  hipLaunchKernelGGL(row, dim3((unsigned)height), dim3(threads), lds, st, a);
  ctx->rec.end(st);
  if (hipGetLastError() != hipSuccess) return fail(ctx, IWPP_EDEVICE, "edt_exact: launch failed");
  ctx->last_stream = st;
  ctx->last_fixed = ctx->fixed;
  ctx->last_op = 2;
  ctx->have_call = false;  // no counters: iwpp_get_stats reports zeros
  return IWPP_OK;
}
