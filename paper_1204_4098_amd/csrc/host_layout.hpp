// Host-side storage layout, batch work lists and the tuner's selection rule of
// the library, in plain C++ (no HIP), so that they can also be built with the
// host sanitizers.  Used by lbm_lib.hip.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <functional>
#include <queue>
#include <utility>
#include <vector>

namespace lbm {

// A tile of the batched launch.  In the balanced schedule an item is a whole
// strip of one run and row0 is its first row in the concatenated row space of
// all items (rows of earlier items summed); in item lists entry b's row0 is the first
// item of block b (deal).
struct Item {
  int32_t run, x0, y0, ncols, nrows, row0;
};

namespace layout {

constexpr int kEX[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int kEY[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

// Population storage, row-interleaved: element (a, y, x) at a * plane + y * rs
// + x with rows of pitch elements (nx rounded up to 64), plane = pitch and rs =
// 9 pitch, so the nine direction rows of one lattice row are consecutive in
// memory.  A row of the march then reads and writes three 9-row blocks close
// together instead of 18 rows in nine planes far apart: on the 4096 x 4096
// FP64 workload a memory-only marching probe reaches 5.5 TB/s against 5.2 with
// plane-major storage (plane = ny pitch, rs = pitch).
inline int pitch_of(int nx) { return (nx + 63) / 64 * 64; }
inline int64_t plane_of(int nx) { return (int64_t)pitch_of(nx); }
inline int64_t rs_of(int nx) { return 9 * (int64_t)pitch_of(nx); }
inline int64_t elems_of(int nx, int ny) { return 9 * (int64_t)pitch_of(nx) * ny; }

// Encode FP64 populations f[a][y][x] (nx*ny per direction) into the
// pre-streamed storage b (elems_of elements, padding left as it is): b holds
// f*_a(x, y) at node (x, y), and the kernel's pull reads it at (x + e_a, y +
// e_a); so b(a, y, x) = f[a][y + ey][x + ex] (periodic).  enc(a, v) converts
// one value to the storage type.
template <typename S, class Enc>
void encode(int nx, int ny, const double* f, S* b, Enc&& enc) {
  const int64_t plane = plane_of(nx), rs = rs_of(nx), n = (int64_t)nx * ny;
  for (int a = 0; a < 9; ++a)
    for (int y = 0; y < ny; ++y) {
      const int ys = (y + kEY[a] + ny) % ny;
      for (int x = 0; x < nx; ++x) {
        const int xs = (x + kEX[a] + nx) % nx;
        b[a * plane + (int64_t)y * rs + x] = enc(a, f[a * n + (int64_t)ys * nx + xs]);
      }
    }
}

// The inverse: dec(a, s) converts one stored value to FP64.
template <typename S, class Dec>
void decode(int nx, int ny, const S* b, double* f, Dec&& dec) {
  const int64_t plane = plane_of(nx), rs = rs_of(nx), n = (int64_t)nx * ny;
  for (int a = 0; a < 9; ++a)
    for (int y = 0; y < ny; ++y) {
      const int ys = (y - kEY[a] + ny) % ny;
      for (int x = 0; x < nx; ++x) {
        const int xs = (x - kEX[a] + nx) % nx;
        f[a * n + (int64_t)y * nx + x] = dec(a, b[a * plane + (int64_t)ys * rs + xs]);
      }
    }
}

// Elements of one run in the batch pool (rounded up to 64).
inline int64_t run_elems(int nx, int ny) { return (elems_of(nx, ny) + 63) / 64 * 64; }

// A launch has fewer than 2^32 threads.
inline bool launchable(int64_t blocks, int threads) { return blocks * threads < (int64_t)1 << 32; }
// Blocks of a launch of nstrips strips in chunks of L rows (0 for the balanced schedule, L = 0).
inline int64_t chunks(int nstrips, int ny, int L) { return L > 0 ? (int64_t)nstrips * ((ny + L - 1) / L) : 0; }
// Square patches (k_patch) of ts steps: nodes along a side, of which 4 ts - 2 are halo, a
// thread a node in whole waves, and blocks.
constexpr int patch_side(int ts) { return ts == 4 ? 22 : 32; }
constexpr int patch_threads(int ts) { return (patch_side(ts) * patch_side(ts) + 63) / 64 * 64; }
inline int patches_across(int n, int ts) {
  const int inner = patch_side(ts) - (4 * ts - 2);
  return (n + inner - 1) / inner;
}
inline int64_t patches(int nx, int ny, int ts) { return (int64_t)patches_across(nx, ts) * patches_across(ny, ts); }

// The most items any offered tile can produce for a run (1 wave, 4 rows).
inline int max_items(int nx, int ny) { return ((nx + 63) / 64) * ((ny + 3) / 4); }

// Work list of a batch tile: per run, chunks of L rows times strips of 64*nw
// columns, or for a multi-step tile (ts > 1) strips of at most 64*nw - (4 ts - 2)
// columns spread evenly over the run's width with their edges rounded down to
// multiples of `align` columns (such items also suit the kernels of fewer steps,
// which run a remainder).  L = 0: whole-height strips with row0 set
// for the balanced schedule.  Returns the rows of all items (the balanced
// schedule's row space).
inline int64_t build_items(int nruns, const int* nx, const int* ny, int nw, int L, int ts,
                           std::vector<Item>& items, int align = 1) {
  items.clear();
  const int SW = 64 * nw, A = ts > 1 ? std::max(1, align) : 1;
  const int M = SW - (4 * ts - 2);  // widest strip of a multi-step tile
  int64_t rows = 0;
  for (int r = 0; r < nruns; ++r) {
    const int Lr = L > 0 ? L : ny[r];
    // strips of at most M columns once their edges are rounded down to A
    const int ns = ts == 1 ? (nx[r] + SW - 1) / SW : nx[r] <= M ? 1 : (nx[r] + M - A) / (M - A + 1);
    auto edge = [&](int k) { return k >= ns ? nx[r] : (int)((int64_t)k * nx[r] / ns) / A * A; };
    for (int y0 = 0; y0 < ny[r]; y0 += Lr)
      for (int sx = 0; sx < ns; ++sx) {
        const int x0 = ts > 1 ? edge(sx) : sx * SW;
        const int x1 = ts > 1 ? edge(sx + 1) : std::min(nx[r], x0 + SW);
        const int n = std::min(Lr, ny[r] - y0);
        items.push_back(Item{r, x0, y0, x1 - x0, n, L > 0 ? 0 : (int32_t)std::min<int64_t>(rows, INT32_MAX)});
        rows += n;
      }
  }
  return rows;
}

// Deal a list of items (chunks) to nblocks blocks of about equal cost, an item's cost
// being its rows plus `fill` (what starting it costs in rows): longest first, each to the
// block with the least so far, or, where every block gets 16 items and more, simply in
// runs of equal count.  The list is reordered block by block and row0 of entry b (b <
// nblocks <= items) becomes the index of block b's first item.  (Dealt in turn, 838
// chunks of 32 rows of a sweep over 256 blocks left the fullest with 212 rows of cost for
// a mean of 155.)
inline void deal(std::vector<Item>& items, int nblocks, int fill) {
  const int n = (int)items.size();
  if (n >= 16 * nblocks) {
    for (int b = 0; b < nblocks; ++b) items[b].row0 = (int32_t)((int64_t)n * b / nblocks);
    return;
  }
  std::vector<int> order(n), block(n), first(nblocks + 1, 0);
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return items[a].nrows > items[b].nrows; });
  using Load = std::pair<int64_t, int>;  // cost so far, block
  std::vector<Load> loads(nblocks);
  for (int b = 0; b < nblocks; ++b) loads[b] = {0, b};
  std::priority_queue<Load, std::vector<Load>, std::greater<Load>> least(std::greater<Load>(), std::move(loads));
  for (int i : order) {
    const Load l = least.top();
    least.pop();
    block[i] = l.second;
    ++first[l.second + 1];
    least.push({l.first + items[i].nrows + fill, l.second});
  }
  for (int b = 0; b < nblocks; ++b) first[b + 1] += first[b];
  std::vector<Item> out(n);
  std::vector<int> at(first.begin(), first.end() - 1);
  for (int i : order) out[at[block[i]]++] = items[i];
  for (int b = 0; b < nblocks; ++b) out[b].row0 = first[b];
  items.swap(out);
}

// The same for short one-step chunks, which cost little to start but share their halo
// rows: the blocks of XCD k (every eighth) walk the k-th part of the list side by side, so
// that neighbouring chunks meet in that XCD's L2.  Sweep of 256 runs, us per step, dealt by
// cost and walked: FP32 2 x 16 34.5 and 32.4, 8 x 16 46.9 and 46.0, 4 x 32 46.9 and 53.8;
// FP64 2 x 16 60.7 and 57.5, 4 x 32 70.1 and 75.5 (waves x rows).  So chunks of fewer than
// kWalkRows rows are walked.
constexpr int kWalkRows = 32;
inline void walk(std::vector<Item>& items, int nblocks) {
  const int n = (int)items.size();
  std::vector<Item> out;
  std::vector<int> first(nblocks);
  out.reserve(n);
  // XCD k has (nblocks + 7 - k)/8 blocks; its part of the list is as large a share, so that
  // no block has two items while another has none
  int before[9] = {};
  for (int k = 0; k < 8; ++k) before[k + 1] = before[k] + ((nblocks + 7 - k) >> 3);
  for (int b = 0; b < nblocks; ++b) {
    const int xcd = b & 7, slots = before[xcd + 1] - before[xcd];
    first[b] = (int)out.size();
    const int lo = (int)((int64_t)n * before[xcd] / nblocks), hi = (int)((int64_t)n * before[xcd + 1] / nblocks);
    for (int i = lo + (b >> 3); i < hi; i += slots) out.push_back(items[i]);
  }
  for (int b = 0; b < nblocks; ++b) out[b].row0 = first[b];
  items.swap(out);
}

// Puts the first item of each block (of a list that was dealt or walked) before the list,
// with its place as row0, and an end: nblocks + 1 entries.  A block without items has its
// successor's place.
inline void add_heads(std::vector<Item>& items, int nblocks) {
  const int n = (int)items.size();
  std::vector<Item> out(nblocks + 1, Item{0, 0, 0, 0, 0, n});
  for (int b = 0; b < nblocks; ++b) {
    const int first = items[b].row0;
    if (first < n) out[b] = items[first];
    out[b].row0 = first;
  }
  out.insert(out.end(), items.begin(), items.end());
  items.swap(out);
}

}  // namespace layout

namespace tuning {

// Index of the fastest of n candidates.  time_one(i) times candidate i
// (milliseconds per lattice step; negative on an error; >= 1e30 to skip it).
// A single pass in candidate order is biased by the GPU's clocks drifting down
// over a long back-to-back run (a kernel trace of the FP64 4096 x 4096 tune
// showed candidates late in the list running up to 40 % slower than the same
// kernels before or after the tune).  So the first pass only shortlists the
// kRefine fastest; they are then timed again in kRefine rounds, each round
// starting one candidate later, so that every finalist is timed once at every
// position of a round, and they are ranked by the sum of those times: a drift
// that grows linearly over the calls then adds the same to every finalist's
// sum.  Returns the index, -1 if every candidate was skipped, or -2 after an
// error.
constexpr int kRefine = 6;
template <class TimeOne>
int pick_best(int n, TimeOne&& time_one) {
  std::vector<std::pair<float, int>> first;
  for (int i = 0; i < n; ++i) {
    const float ms = time_one(i);
    if (ms < 0) return -2;
    if (ms < 1e30f) first.push_back({ms, i});
  }
  if (first.empty()) return -1;
  std::sort(first.begin(), first.end());
  const int m = std::min<int>(kRefine, (int)first.size());
  if (m == 1) return first[0].second;
  std::vector<double> sum(m, 0.0);
  for (int r = 0; r < m; ++r)
    for (int q = 0; q < m; ++q) {
      const int k = (q + r) % m;
      const float ms = time_one(first[k].second);
      if (ms < 0) return -2;
      sum[k] += ms;
    }
  int kb = 0;
  for (int k = 1; k < m; ++k)
    if (sum[k] < sum[kb]) kb = k;
  return first[kb].second;
}

}  // namespace tuning
}  // namespace lbm
