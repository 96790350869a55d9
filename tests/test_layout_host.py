"""Dealing of a batch work list to blocks (csrc/host_layout.hpp), compiled for the
host: every item kept once and, dealt by cost, every block at least one and (below 16
items per block) the fullest block at most one item above the mean cost."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "host_layout.hpp"
using namespace lbm;
int main() {
  unsigned seed = 1;
  auto rnd = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
  for (int trial = 0; trial < 300; ++trial) {
    std::vector<int> nx(1 + rnd(60)), ny(nx.size());
    for (size_t i = 0; i < nx.size(); ++i) nx[i] = 3 + rnd(600), ny[i] = 3 + rnd(80);
    const int ts[] = {1, 2, 4};
    std::vector<Item> items;
    layout::build_items((int)nx.size(), nx.data(), ny.data(), 2 + rnd(2), 4 + rnd(60), ts[rnd(3)], items, 8);
    const std::vector<Item> before = items;
    const int n = (int)items.size(), blocks = 1 + rnd(n < 256 ? n : 256), fill = rnd(22);
    const bool walk = trial % 3 == 0;
    if (walk) layout::walk(items, blocks);
    else layout::deal(items, blocks, fill);
    if ((int)items.size() != n) return 1;
    std::vector<char> seen(n, 0);
    long total = 0, most = 0, longest = 0;
    for (int b = 0; b < blocks; ++b) {
      const int lo = items[b].row0, hi = b + 1 < blocks ? items[b + 1].row0 : n;
      if (lo < 0 || hi < lo || (hi == lo && !walk) || hi > n) return 2;
      long cost = 0;
      for (int i = lo; i < hi; ++i) {
        const Item& a = items[i];
        int k = 0;
        while (k < n && (seen[k] || a.run != before[k].run || a.x0 != before[k].x0 || a.y0 != before[k].y0 ||
                         a.ncols != before[k].ncols || a.nrows != before[k].nrows)) ++k;
        if (k == n) return 3;
        seen[k] = 1;
        cost += a.nrows + fill;
        if (a.nrows + fill > longest) longest = a.nrows + fill;
      }
      total += cost;
      if (cost > most) most = cost;
    }
    // many items are dealt by count alone: a few more of the longest than the mean has
    if (!walk && n < 16 * blocks && most > total / blocks + longest) return 4;
  }
  std::puts("ok");
  return 0;
}
"""


def test_deal_keeps_every_item_and_balances(tmp_path):
    src, exe = tmp_path / "deal.cpp", tmp_path / "deal"
    src.write_text(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1204_4098_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out


HEADS = r"""
#include <cstdio>
#include "host_layout.hpp"
using namespace lbm;
int main() {
  unsigned seed = 7;
  auto rnd = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
  for (int trial = 0; trial < 300; ++trial) {
    std::vector<int> nx(1 + rnd(40)), ny(nx.size());
    for (size_t i = 0; i < nx.size(); ++i) nx[i] = 3 + rnd(600), ny[i] = 3 + rnd(80);
    std::vector<Item> items;
    layout::build_items((int)nx.size(), nx.data(), ny.data(), 1 + rnd(3), 4 + rnd(60), 1, items);
    const int n = (int)items.size(), blocks = 1 + rnd(n < 300 ? n : 300);
    if (trial % 2) layout::walk(items, blocks);
    else layout::deal(items, blocks, rnd(22));
    std::vector<Item> list = items;
    layout::add_heads(list, blocks);
    if ((int)list.size() != blocks + 1 + n) return 1;
    int at = 0;  // every item once, in the order of the blocks
    for (int b = 0; b < blocks; ++b) {
      const int first = list[b].row0, end = list[b + 1].row0;
      if (first != at || end < first || end > n) return 2;
      for (int i = first; i < end; ++i, ++at) {
        const Item &a = i == first ? list[b] : list[blocks + 1 + i], &q = items[i];
        if (a.run != q.run || a.x0 != q.x0 || a.y0 != q.y0 || a.ncols != q.ncols || a.nrows != q.nrows) return 3;
      }
    }
    if (at != n) return 4;
  }
  std::puts("ok");
  return 0;
}
"""


def test_first_items_of_blocks(tmp_path):
    src, exe = tmp_path / "heads.cpp", tmp_path / "heads"
    src.write_text(HEADS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined", "-I",
                    os.path.join(ROOT, "paper_1204_4098_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out


WALK = r"""
#include <cstdio>
#include "host_layout.hpp"
using namespace lbm;
int main() {
  for (int n = 1; n < 400; ++n)
    for (int blocks : {n, (n + 1) / 2, (n + 2) / 3}) {
      std::vector<Item> items(n);
      for (int i = 0; i < n; ++i) items[i] = Item{i, 0, 0, 1, 8, 0};
      layout::walk(items, blocks);
      for (int b = 0; b < blocks; ++b) {
        const int k = (b + 1 < blocks ? items[b + 1].row0 : n) - items[b].row0;
        if (k > (n + blocks - 1) / blocks + (blocks < n)) return 1;   // one each where there are as many
        if (blocks == n && k != 1) return 2;
      }
    }
  std::puts("ok");
  return 0;
}
"""


def test_walk_gives_no_block_two_items_and_another_none(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined", "-I",
                    os.path.join(ROOT, "paper_1204_4098_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out


LAUNCH = r"""
#include <cstdio>
#include "host_layout.hpp"
using namespace lbm::layout;
int main() {
  // patches: 8, 26 and 22 nodes stored of 22, 32 and 32
  if (patches(64, 32, 4) != 8 * 4 || patches(65, 33, 4) != 9 * 5 || patches(26, 27, 2) != 2 || patches(23, 22, 3) != 2) return 1;
  if (patch_threads(4) != 512 || patch_threads(3) != 1024 || patch_threads(2) != 1024) return 2;
  // 512 threads for 64 nodes: 2^29 nodes are too many, one row of patches less is not
  if (launchable(patches(16384, 32768, 4), 512) || !launchable(patches(16384, 32760, 4), 512)) return 3;
  if (launchable(patches(46340, 46340, 4), 512) || !launchable(patches(46340, 46340, 2), 1024)) return 4;
  // 768 threads for a strip of three columns and one row
  if (launchable(chunks(1, 5592406, 1), 768) || !launchable(chunks(1, 5592405, 1), 768)) return 5;
  if (!launchable(chunks(1, 700000000, 0), 768) || chunks(3, 10, 4) != 9) return 6;
  std::puts("ok");
  return 0;
}
"""


def test_launches_of_fewer_than_2_to_the_32_threads(tmp_path):
    src, exe = tmp_path / "launch.cpp", tmp_path / "launch"
    src.write_text(LAUNCH)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=address,undefined", "-I",
                    os.path.join(ROOT, "paper_1204_4098_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out
