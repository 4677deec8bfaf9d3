"""Host-checkable headers of the kernels, compiled with g++.

The schedule's integer arithmetic (csrc/sla_items.h): every wave of every item gets a
head of the tensor, also where it is idle (kernels index per-head arrays with it), and
every share of a long window and every part of a chunk is some wave's exactly once.

The table of launch figures (csrc/sla_cache.h) under the thread sanitizer: threads
that look up the same and different kernels for the first time."""
from __future__ import annotations

import subprocess

import pytest

from paper_2401_00912_amd.build import CSRC

HARNESS = r"""
#include "sla_items.h"
#include <cstdio>
#include <map>
#include <tuple>
using namespace sla;
int main() {
  const int heads[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 16}, longs4[] = {0, 1, 9}, longs2[] = {0, 5, 8};
  const int chunks[] = {0, 1, 3, 17, 64}, grids[] = {8, 512}, fills[] = {0, 100, 400};
  for (int H : heads) for (int nL4 : longs4) for (int nL2 : longs2) for (int nC : chunks)
  for (int grid : grids) for (int fill : fills) {
    const Items it = make_items(nL4, nL2, nC, H, 200, grid, fill, kMaxPartBits);
    std::map<std::tuple<int, int, int, int>, int> seen;
    for (int item = 0; item < it.total + 2 * grid; ++item)
      for (int wv = 0; wv < 4; ++wv) {
        const Slot s = item_slot(it, item, wv);
        if (s.h < 0 || s.h >= H) {
          std::printf("H=%d nL4=%d nL2=%d nC=%d grid=%d item=%d wave=%d: head %d\n", H, nL4, nL2, nC, grid, item, wv, s.h);
          return 1;
        }
        if (s.idx < 0 || s.piece < 0) continue;
        if (s.idx >= (s.table == 0 ? nL4 + nL2 : nC)) return 2;
        if (s.table == 0 && s.parts != (s.idx < nL4 ? 4 : 2)) return 3;
        ++seen[std::make_tuple(s.table, s.idx, s.h, s.table == 0 ? s.piece : s.part)];
      }
    if ((int)seen.size() != H * (4 * nL4 + 2 * nL2 + (nC << it.part_bits))) return 4;
    for (const auto& e : seen)
      if (e.second != 1) return 5;
  }
  return 0;
}
"""

TABLE = r"""
#include "sla_cache.h"
#include <cstdio>
#include <thread>
#include <vector>
int main() {
  static sla::LaunchTable<32> table;   // smaller than the keys below: the rest is computed each time
  static char kernels[24];
  std::vector<std::thread> threads;
  std::atomic<int> wrong{0};
  for (int t = 0; t < 8; ++t)
    threads.emplace_back([&, t] {
      for (int round = 0; round < 200; ++round)
        for (int k = 0; k < 24; ++k)
          for (int dev = 0; dev < 2; ++dev) {
            const int key = (k + 3 * t) % 24, want = 256 * (key + 1) + dev;
            if (table.get(&kernels[key], dev, [&] { return want; }) != want) ++wrong;
          }
    });
  for (auto& th : threads) th.join();
  return wrong.load() ? 1 : 0;
}
"""


@pytest.fixture(scope="module")
def gxx(tmp_path_factory):
    """Compile a harness against the kernels' host-checkable headers and run it."""
    def run(source, *flags, wrap=()):
        out = tmp_path_factory.mktemp("items")
        (out / "harness.cc").write_text(source)
        exe = str(out / "harness")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-D__host__=", "-D__device__=",
                        "-D__forceinline__=inline", "-I", CSRC, *flags, str(out / "harness.cc"), "-o", exe],
                       check=True, capture_output=True, text=True)
        return subprocess.run([*wrap, exe], capture_output=True, text=True, timeout=120)
    return run


def test_every_wave_has_a_head_and_every_share_a_wave(gxx):
    res = gxx(HARNESS)
    assert res.returncode == 0, (res.returncode, res.stdout)


def test_launch_table_is_safe_with_threads(gxx):
    # (address randomisation off: the sanitizer's shadow needs the low mappings free)
    res = gxx(TABLE, "-g", "-pthread", "-fsanitize=thread", wrap=["setarch", "-R"])
    assert res.returncode == 0, (res.returncode, res.stdout, res.stderr[-2000:])


PARTS = r"""
#include "sla_items.h"
#include <cstdio>
using namespace sla;
int main() {
  // where the host takes the kernels with parts, the device splits the chunks of a scene of
  // the guessed size, and nowhere else; parts fill the grid as far as they may
  const int heads[] = {1, 2, 3, 4, 6, 8, 12}, windows[] = {38, 169, 900, 1521, 3481}, grids[] = {512, 768, 1536};
  const int fills[] = {100, 200, 400};
  int with = 0, without = 0;
  for (int H : heads) for (int W : windows) for (int grid : grids)
  for (int n = 50; n < 300000; n = n * 5 / 4) {
    int nC = (n + kThinChunkRows - 1) / kThinChunkRows;
    if (nC > W) nC = W;
    for (int fill : fills) {
      const Items it = make_items(0, 0, nC, H, W, grid, fill, kMaxPartBits);
      if ((it.part_bits > 0) != parts_fit(grid, n, W, H, fill)) return 1;
      if (it.part_bits > 0 && it.total > fill * (long)grid / 100) return 2;
    }
    const int bits = proj_part_bits(nC, H, W, grid);
    if ((bits > 0) != proj_parts_fit(grid, n, W, H)) return 3;
    if (bits > 0 && (((long)(nC + 3) / 4) << bits) * H > grid) return 4;
    if (bits > 0 && ((long)nC << bits) > W) return 5;
    ++(bits > 0 ? with : without);
  }
  // 16k rows in 3,481 windows, 8 heads: 498 chunks fill the projection's grid without parts
  if (proj_parts_fit(512, 16001, 3481, 4)) return 6;
  return with > 50 && without > 50 ? 0 : 7;
}
"""


def test_parts_where_the_device_splits(gxx):
    res = gxx(PARTS)
    assert res.returncode == 0, res.returncode
