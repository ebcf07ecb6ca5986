// Internal declarations shared by the host library and the kernel sources.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace iwpp {

struct GridBarrier;

// Tile geometry shared by the host plans and the kernels.
constexpr int kMrTile = 64;   // reconstruction tiles: 64 x 64 pixels
constexpr int kEdtHalo = 8;   // EDT rounds per tile visit (= halo width)
constexpr int kEdtTile = 48;  // EDT tiles: 48 x 48 pixels (a 64 x 64 region with the halo)
// EDT change records: for every column of tiles one run of row words, a bit per
// pixel of the row in that column; a narrow last column takes shorter words, and
// there are no more rows than the image has.  (48 words of 8 bytes a tile whatever
// its size would be 16 bytes a row of an image one pixel wide, where this is 2.)
constexpr int edt_mark_shift(int cols) { return cols > 32 ? 3 : (cols > 16 ? 2 : (cols > 8 ? 1 : 0)); }
// 8-byte words of an image's records, with one more: words are read as 8 bytes each.
constexpr uint64_t edt_mark_words(int32_t h, int32_t w) {
  const int32_t full = (w - 1) / kEdtTile;  // tile columns before the last
  return (uint64_t)full * (uint64_t)h + (((uint64_t)h << edt_mark_shift(w - full * kEdtTile)) + 7) / 8 + 1;
}
constexpr size_t kEdtStatePad = 256;  // bytes after each EDT state buffer (16-byte loads may cross the end)

// One reconstruction image of a launch.
struct MrJob {
  const uint8_t* marker;
  const uint8_t* mask;
  uint8_t* out;
  int32_t h, w;
  int32_t tiles_y, tiles_x;
  uint32_t tile_base;  // first global tile id of this image
  // 0 for reconstruction by dilation; all ones for reconstruction by
  // erosion, computed as the dilation of the complemented images (every
  // image byte is complemented as it is loaded and stored).
  uint32_t inv;
};

// Reconstruction launch arguments (device pointers, scratch owned by the context).
// A launch processes njobs images; global tile ids run over all of them.
struct MrArgs {
  MrJob job0;                // the image when njobs == 1 (no table lookup)
  const MrJob* jobs;         // [njobs] device table when njobs > 1
  uint32_t* tile_job;        // [ntiles] image of each global tile when njobs > 1
  uint32_t njobs;
  uint32_t ntiles;           // total tiles over all images
  uint32_t list_cap;         // capacity of each round's tile list (<= ntiles)
  int32_t max_sweeps;        // sweep iterations per propagation visit before re-listing
  int32_t seed_sweeps;       // sweep iterations per tile in the seed pass
  uint32_t seed_only;        // nonzero: stop after the seed pass (round 0)
  uint32_t seed_strip;       // seed pass: tiles per strip (0 = automatic)
  uint32_t stage_depth;      // work-list items staged per wave before a flush (0 = the LDS maximum)
  uint32_t wg_waves;         // waves per workgroup: 4 or 8
  uint32_t* flags;           // [2][ntiles] tile on the round's list, per round parity
  uint32_t* lists;           // [2][8 shards][ntiles] tile lists per round parity
  uint32_t* unsettled;       // [ntiles] the tile's last visit stopped at the sweep cap
  uint8_t* cols;             // [ntiles][4][64] each tile's border columns: J left, J right, I left, I right
  uint32_t* counts;          // [3 round slots][8 shards][64] list fill levels (256 B apart)
  uint32_t* lost;            // [2][64] a listed tile was dropped (capacity), per parity
  GridBarrier* bar;
  unsigned long long* stats;  // [8 shards][16 fields]
  unsigned long long* clock;  // [kClockWords] round timeline (see kClockWords)
};

// One distance-transform image of a launch.
struct EdtJob {
  const uint8_t* bin;
  int32_t* sqdist;
  int32_t* nearest;
  int32_t h, w;
  int32_t tiles_y, tiles_x;  // kEdtTile x kEdtTile tiles
  uint32_t tile_base;        // first global tile id of this image
  uint32_t mark_base;        // first word of this image's change records
  unsigned long long pix_base;  // first global pixel id of this image
};

// Distance-transform launch arguments.  Global pixel id = pix_base + y*w + x;
// global tile ids run over all images.
struct EdtArgs {
  EdtJob job0;                // the image when njobs == 1
  const EdtJob* jobs;         // [njobs] device table when njobs > 1
  uint32_t* tile_job;         // [ntiles] image of each global tile when njobs > 1
  uint32_t njobs;
  uint32_t ntiles;
  uint32_t wide;              // nonzero: wide coordinate fields (an image side above 32767)
  uint32_t mark_words;        // 8-byte words of change records of all images (one step parity)
  unsigned long long npix;    // total pixels over all images
  uint32_t* feat0;            // [npix] nearest feature (y << 16 | x), ~0 = none; round parity 0
  uint32_t* feat1;            // [npix] round parity 1
  uint32_t* flags;            // [2][ntiles] tile on the round's list, per round parity
  uint32_t* lists;            // [2][8 shards][ntiles] tile lists per round parity
  uint32_t* stamps;           // [2][ntiles] step of the tile's last visit, per step parity (0 = none)
  unsigned long long* marks;  // [2][mark_words] that visit's last-round changes (see edt_mark_words)
  uint32_t* counts;           // [3 round slots][8 shards][64] list fill levels (256 B apart; word 32: items taken)
  uint32_t* ovf;              // never set: a list holds each tile once
  uint32_t stage_depth;       // work-list items staged per wave before a flush (0 = the LDS maximum)
  uint32_t wg_waves;          // waves per workgroup of the rounds kernel: 4, 8 or 0 = automatic (edt_waves)
  GridBarrier* bar;
  unsigned long long* stats;
  unsigned long long* clock;  // [kClockWords] round timeline (see kClockWords)
};

// Bytes of the scratch areas the kernels expect.
constexpr size_t kBarrierBytes = 4096;
constexpr size_t kCountsBytes = 3 * 8 * 64 * 4;
// Round timeline: word 0 = stamps written, words 1..255 realtime-clock stamps
// (kernel start, then after every grid barrier) of one workgroup, words
// 256 + i the tiles visited in phase i.
constexpr int kClockWords = 512;
constexpr size_t kLostBytes = 2 * 64 * 4;
constexpr size_t kStatsBytes = 8 * 16 * 8;

// Waves per workgroup of the persistent kernels (iwpp_options.wg_waves, 0 =
// automatic).  A caller that caps the workgroups (iwpp_options.persistent_blocks)
// has sized its cap for four waves each, so the automatic choice is four then: with
// eight, half the device would have become all of it.
//
// Reconstruction, eight waves: twice as many take tiles from one workgroup's
// share, and half as many workgroups meet at the barrier (us with 4, 8: 16384^2
// 1456, 1374 and with 4-connectivity 1431, 1347; 4096^2 269, 258; 65536 x 65600
// 12880, 12200; 1500 x 1301 154, 149; 512^2 114, 114).  The 1% lost at 20000 x 17000
// (1868, 1895) is its strips' (see `auto_strip`): seeded by single tiles it takes 1736.
constexpr uint32_t recon_waves(int32_t wg_waves, int32_t persistent_blocks) {
  return wg_waves == 4 || (wg_waves == 0 && persistent_blocks > 0) ? 4u : 8u;
}
// Distance transform: a workgroup's waves share a tile.  `cus`: the device's compute
// units, each of which holds two workgroups of eight waves.  Where every tile of the
// launch has such a workgroup a visit is shorter with eight waves (30% features with
// 8-connectivity, 15%, 30% with 4-connectivity; us with 4 and 8 waves: 400 tiles 382
// 346, 648 560, 388 368; 512 tiles 342 319, 526 480, 358 346).  Past that some
// workgroups visit two tiles a step; up to 20% more tiles eight waves still gain with
// few features and lose with 4-connectivity (576 tiles 417 401, 632 569, 394 424; 600
// tiles 417 426, 506 462, 414 441), and with many more tiles four workgroups of four
// hide more (1024 tiles 402 467, 625 666, 423 523).
constexpr uint32_t edt_waves(int32_t wg_waves, int32_t persistent_blocks, uint64_t ntiles, int cus) {
  return wg_waves == 8 || (wg_waves == 0 && persistent_blocks == 0 && ntiles <= 2u * (uint64_t)cus) ? 8u : 4u;
}

// Optional per-launch event timing (iwpp_options.profile).  begin/end bracket
// one kernel launch on `s`; both are no-ops when disabled or full.
class Recorder {
 public:
  static constexpr int kCap = 4096;
  bool enabled = false;
  void begin(int kernel, hipStream_t s);
  void end(hipStream_t s);
  // Completed records since the last read: returns the count written.
  int read(int* kernels, float* ms, int max);
  void release();

 private:
  hipEvent_t start_[kCap] = {};
  hipEvent_t stop_[kCap] = {};
  int kernel_[kCap] = {};
  int created_ = 0;
  int count_ = 0;
  bool open_ = false;
};

int mr_launch(const MrArgs& a, int conn, int persistent_blocks, hipStream_t stream, Recorder* rec, const char** err);
int edt_launch(const EdtArgs& a, int conn, int persistent_blocks, hipStream_t stream, Recorder* rec, const char** err);
int zero_words(uint32_t* p, size_t nwords, hipStream_t stream, uint32_t* q = nullptr, size_t mwords = 0);

// Workgroups for a cooperative (persistent) launch of `fn`: every one must be
// resident at once, since they meet at grid barriers.  The runtime's occupancy
// figure is capped by the 160 KiB of LDS of a CU and by `max_per_cu`
// workgroups per CU (4 unless the kernel's registers and LDS fit more); grids
// sized from the raw figure (8 per CU for a 16 KiB kernel) were measured not
// to be co-resident on MI355X, while these caps are.
uint32_t persistent_grid(const void* fn, int per_cu, int cus, int max_per_cu = 4);

// Launch a persistent kernel: a cooperative launch (the runtime checks that the
// whole grid is resident), or a plain launch of the same grid while `s` is being
// captured into a graph.  Inside a graph, residency then rests on the grid
// fitting the device when the graph runs alone; a grid that does not fit makes
// the grid barrier time out and report an error instead of waiting forever.
hipError_t launch_persistent(const void* fn, uint32_t blocks, void** args, hipStream_t s, uint32_t threads = 256);

}  // namespace iwpp
