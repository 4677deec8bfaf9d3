// Work items of a launch and the wave that takes each: the integer arithmetic of the
// attention and XCA kernels' schedule.  No HIP header is needed, so that it can be
// compiled and checked on the host.
#pragma once
#include <stdint.h>

namespace sla {

constexpr int32_t kMaxChunkRows = 64;   // rows one wavefront holds in registers
constexpr int kMaxPartBits = 4;

// ------------------------------------------------------------- work items
// A launch walks a list of work items; workgroup b takes items b, b + G, ...
// (G = grid size, a multiple of 8, about the number of resident workgroups).
// In order:
//   long items   one per (long window, head): the four waves of the workgroup
//                take a quarter of the window's rows each, add their partial
//                states in LDS (in wave order, so every wave holds the same sum)
//                and then form their rows' outputs.  Item numbers are laid out so
//                that the heads of one window share an item residue mod 8, i.e.
//                run on one XCD (workgroups are dealt to the 8 XCDs round-robin),
//                where the L2 serves the other heads' halves of each row.
//   chunk items  one per chunk and group of up to 4 heads (one wave per head;
//                with fewer than 4 heads, several chunks share a workgroup).
//                A scene whose items do not fill the grid splits every chunk into
//                2^part_bits items, each of which takes a share of its non-empty
//                windows and reads their rows only: a chunk of thin windows is a
//                serial chain of up to 32 of them on one wave while the rest of the
//                chip idles.  fp16 forward + backward (with the build), 1,521
//                windows: 2k rows 110 -> 42 us, 6k rows 76 -> 56 us; fp32 forward of
//                1.9k rows in 64 windows 15.0 -> 12.0 us.  There are at most as many
//                parts as window slots, twice that where they fill an eighth of the
//                grid (at a third, 6k rows in 200 windows, it cost 16.5 -> 17.3 us).
// Long items come first: they are the longest-running ones.
//
// Each wave software-pipelines its items: while item k computes, the plan entry
// of item k + 2 and the permutation entries and window offsets of item k + 1 are
// in flight, so an item's row gathers start as soon as the previous item's rows
// have been requested and its data path is one memory round trip long.
struct Items {
  int32_t nL4, nL2, nC, H, hp, hw, cpw, hg;
  int32_t itemsL4, itemsL, total;
  int32_t part_bits;
};

// nL4 four-way and nL2 two-way long windows, nC chunks on a grid of `grid` workgroups.
// fill: how many times the grid (in percent) the parts may fill; 0: no parts.
__host__ __device__ __forceinline__ Items make_items(int32_t nL4, int32_t nL2, int32_t nC, int32_t H, int32_t W,
                                                     int32_t grid, int fill, int bits) {
  Items it;
  it.nL4 = nL4;
  it.nL2 = nL2;
  it.nC = nC;
  it.H = H;
  it.hp = (H + 1) / 2;
  it.hw = H < 4 ? H : 4;
  it.cpw = 4 / it.hw;
  it.hg = (H + 3) / 4;
  it.itemsL4 = ((it.nL4 + 7) & ~7) * H;
  it.itemsL = it.itemsL4 + ((it.nL2 + 7) & ~7) * it.hp;
  const int32_t chunks = (it.nC + it.cpw - 1) / it.cpw * it.hg;
  it.part_bits = 0;
  while (fill > 0 && it.part_bits < bits) {
    const int64_t items = (int64_t)chunks << (it.part_bits + 1);
    if (items > fill * (int64_t)grid / 100) break;
    // parts without a window are cheap only while most of the grid is idle
    const int64_t parts = (int64_t)it.nC << (it.part_bits + 1);
    if (parts > (items <= (int64_t)grid / 8 ? 2 : 1) * (int64_t)W) break;
    ++it.part_bits;
  }
  it.total = it.itemsL + (chunks << it.part_bits);
  return it;
}

// Where item `item` puts wave wv (wave-uniform): table entry index (-1: none),
// the table (0: long windows, 1: chunks), the head (always one of the tensor's,
// also for an idle wave: kernels index per-head arrays with it), and for a long window how
// many waves share it and which share is this wave's (-1: none, the wave only
// takes part in the workgroup's partial-state exchange).
//   four-way long items: one per (window, head), the four waves take quarters;
//   two-way long items: one per (window, pair of heads), waves 2m and 2m + 1
//     take the halves of head 2 x (item's pair) + m.
struct Slot {
  int32_t idx;
  int table, h, parts, piece, part;
};

__host__ __device__ __forceinline__ Slot item_slot(const Items& it, int32_t item, int wv) {
  Slot sl;
  sl.idx = -1;
  sl.table = 0;
  sl.h = 0;
  sl.parts = 4;
  sl.piece = wv;
  sl.part = 0;
  if (item >= it.total) return sl;
  if (item < it.itemsL4) {
    const int32_t r = item >> 3;
    const int32_t j = (r / it.H) * 8 + (item & 7);
    sl.h = r % it.H;
    if (j < it.nL4) sl.idx = j;
  } else if (item < it.itemsL) {
    const int32_t r = (item - it.itemsL4) >> 3;   // itemsL4 is a multiple of 8
    const int32_t j = (r / it.hp) * 8 + (item & 7);
    const int h = (r % it.hp) * 2 + (wv >> 1);
    sl.parts = 2;
    sl.piece = h < it.H ? (wv & 1) : -1;
    sl.h = h < it.H ? h : 0;
    if (j < it.nL2) sl.idx = it.nL4 + j;
  } else {
    const int32_t bp = item - it.itemsL, b = bp >> it.part_bits;
    sl.part = bp - (b << it.part_bits);
    const int32_t grp = b / it.hg;
    const int sub = wv / it.hw;
    const int32_t c = grp * it.cpw + sub;
    sl.table = 1;
    const int h = (b - grp * it.hg) * 4 + wv % it.hw;
    sl.h = h < it.H ? h : 0;
    if (sub < it.cpw && c < it.nC && h < it.H) sl.idx = c;
  }
  return sl;
}

// Rows of a chunk, as the host guesses their number before the plan is there: windows of up
// to 32 rows share one when they start in the same 32 rows of the sorted order, so a scene of
// thin windows has chunks of 32 to 35 rows (frames of 6k to 16k rows in 900 to 3,481
// windows), one of 60k rows in 1,521 windows 62.
constexpr int32_t kThinChunkRows = 36;

// Whether a launch of `grid` workgroups will split its chunks into parts, by that guess and
// the rule of make_items.  The kernels without parts, two to four percent faster where
// nothing is split, run otherwise.
inline bool parts_fit(int grid, int32_t n, int32_t W, int32_t H, int fill) {
  const int32_t chunks = (n + kThinChunkRows - 1) / kThinChunkRows;
  return make_items(0, 0, chunks < W ? chunks : W, H, W, grid, fill, 1).part_bits > 0;
}

// The same for the fused projection: nC chunks, four to a workgroup of every head, split into
// 2^bits parts that fill the grid at most once.
__host__ __device__ __forceinline__ int proj_part_bits(int32_t nC, int32_t H, int32_t W, int32_t grid) {
  const int64_t groups = ((int64_t)nC + 3) / 4;
  int bits = 0;
  while (bits < kMaxPartBits && ((int64_t)nC << (bits + 1)) <= W && (groups << (bits + 1)) * H <= grid) ++bits;
  return bits;
}

inline bool proj_parts_fit(int grid, int32_t n, int32_t W, int32_t H) {
  const int32_t chunks = (n + kThinChunkRows - 1) / kThinChunkRows;
  return proj_part_bits(chunks < W ? chunks : W, H, W, grid) > 0;
}

}  // namespace sla
