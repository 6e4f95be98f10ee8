// Work list of the pair kernels for one launch over all cells of uneven
// occupancy (Alg. 1 CallQuadratic): one item per chunk of at most ti
// consecutive slots of a cell, the cells in brick order (brick_cell). The
// items are split into 8 contiguous ranges, one per XCD, so neighbouring
// cells are processed on the same XCD and share its L2. The ranges balance
// an estimated cost rather than the item count: a chunk of a cell costs
// about (its particle count) x (the particle count of the 27 cells around
// it, capped at 27 x 64) candidate tests, so a few crowded cells weigh as
// much as many sparse ones. Each item writes only its own particles'
// outputs, so no result depends on the split, the order or the schedule.
//
// Buffer layout: [0, kWorkHeader) queue counters[8] and meta (item count,
// range boundaries[9]); then the prefixes of the items and of the costs of
// the cells in brick order ([C + 1] each, see k_wl_count) and the items (int2:
// cell, first slot).
//
// Two launches: the lists are short (a few us of work), so what a build costs
// is its launches. With separate scans of items and costs and a kernel for the
// boundaries, nine launches, it took 37 us for 4096 cells and 59 us for
// 287496; now 13 and 30.
#include <algorithm>

#include "sph_device.h"

namespace sph {
namespace {

constexpr int kThreads = 256;
constexpr int kCostShift = 12;   // cost unit: 4096 candidate tests
constexpr int kNbCap = 27 * 64;  // neighbour-count cap of the cost estimate

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

struct WlLayout {
  int32_t* pos;       // [C + 1] item prefixes of the cells (brick order)
  int32_t* cost;      // [C + 1] cost prefixes of the cells (brick order)
  int2* items;
};

size_t al256(size_t b) { return (b + 255) & ~size_t(255); }

WlLayout wl_layout(void* buf, int C) {
  char* p = static_cast<char*>(buf) + kWorkHeader;
  WlLayout L;
  L.pos = reinterpret_cast<int32_t*>(p);
  p += al256(sizeof(int32_t) * ((size_t)C + 1));
  L.cost = reinterpret_cast<int32_t*>(p);
  p += al256(sizeof(int32_t) * ((size_t)C + 1));
  L.items = reinterpret_cast<int2*>(p);
  return L;
}

__device__ __forceinline__ int cell_count(const int32_t* __restrict__ start, int c, int n) {
  const int a = min(max(start[c], 0), n);
  return max(min(max(start[c + 1], 0), n) - a, 0);
}

// Merged items: in a launch over an occupancy class, consecutive non-empty
// cells of the class along x within one row of a brick (bricks are 4 cells
// wide) are grouped greedily from the row's first cell, up to `merge` cells
// whose particles fit one tile; a cell outside the class, an empty cell or
// a cell with more than ti particles ends a group and is not merged. The
// group's first cell carries one item for all of its slots (a contiguous
// slot range: cells of a row are consecutive in id order); the others carry
// none. Returns the group size m of cell c's group if c starts one (1 for an
// unmerged cell), 0 if c is inside a group started by another cell.
__device__ __forceinline__ int merge_group(const int32_t* __restrict__ start, int n, int n_c,
                                           int ti, int merge, int occ_lo, int occ_hi, int c) {
  int cx, cy, cz;
  cell_coords(c, n_c, cx, cy, cz);
  const int x0 = cx - cx % kBrick, tx = min(kBrick, n_c - x0);
  int rc[kBrick];
#pragma unroll
  for (int l = 0; l < kBrick; ++l) {
    int k = -1;
    if (l < tx) {
      k = cell_count(start, (x0 + l) + n_c * (cy + n_c * cz), n);
      if (k <= 0 || k < occ_lo || k >= occ_hi || k > ti) k = -1;   // not mergeable
    }
    rc[l] = k;
  }
  int l = 0;
  while (l < tx) {
    int m = 1;
    if (rc[l] > 0) {
      int sum = rc[l];
      while (l + m < tx && m < merge && rc[l + m] > 0 && sum + rc[l + m] <= ti) sum += rc[l + m++];
    }
    if (cx - x0 == l) return m;
    if (cx - x0 < l + m) return 0;
    l += m;
  }
  return 1;
}

// Cells of a block: `rounds` times kThreads, so that at most kMaxBlocks blocks
// hold all cells and every block can add up the totals of those before it.
constexpr int kMaxBlocks = 4 * kThreads;
int wl_rounds(int C) { return std::max(cdiv(C, kThreads * kMaxBlocks), 1); }

// items << 32 | cost of a range of cells: both sums stay below 2^31
__device__ __forceinline__ uint64_t pair64(int items, int cost) {
  return (uint64_t)(uint32_t)items << 32 | (uint32_t)cost;
}
__device__ __forceinline__ int items_of(uint64_t v) { return (int)(v >> 32); }
__device__ __forceinline__ int cost_of(uint64_t v) { return (int)(uint32_t)v; }

// Exclusive prefix of v over the block; `total`: the block's sum
__device__ __forceinline__ uint64_t block_prefix(uint64_t v, uint64_t& total, uint64_t* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t t = __shfl_up(inc, o);
    inc += lane >= o ? t : 0;
  }
  if (lane == 63) lds[wave] = inc;
  __syncthreads();
  uint64_t pre = inc - v;
  total = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    pre += w < wave ? lds[w] : 0;
    total += lds[w];
  }
  __syncthreads();
  return pre;
}

// Particles in the cells x - 1 .. x + 1 of a row (the row's first cell: row)
__device__ __forceinline__ int row_count(const int32_t* __restrict__ start, int n_c, int n,
                                         int row, int cx) {
  auto slot = [&](int c) { return min(max(start[c], 0), n); };
  if (cx > 0 && cx + 1 < n_c) return max(slot(row + cx + 2) - slot(row + cx - 1), 0);
  int k = 0;
  for (int dx = -1; dx <= 1; ++dx)
    k += cell_count(start, row + (cx + dx + n_c) % n_c, n);
  return k;
}

// Items per cell and the cell's cost estimate, clamped so that the sum over
// all cells fits in int32, as exclusive prefixes within the block's cells. The
// first cell of a block, whose prefix is zero, holds the block's total instead.
__global__ __launch_bounds__(kThreads) void k_wl_count(const int32_t* __restrict__ start, int n_c,
                                                        int n, int ti, int cost_cap, int rounds,
                                                        const uint8_t* __restrict__ active,
                                                        int occ_lo, int occ_hi, int merge,
                                                        int32_t* __restrict__ pos,
                                                        int32_t* __restrict__ cost,
                                                        const int32_t* gate) {
  __shared__ uint64_t lds[kThreads / 64];
  if (gate && *gate == 0) return;             // the cell list was kept: so is this list
  const int C = n_c * n_c * n_c;
  const int j0 = blockIdx.x * (rounds * kThreads);
  uint64_t carry = 0;
  for (int r = 0; r < rounds; ++r) {
    const int j = j0 + r * kThreads + threadIdx.x;   // position in brick order
    int items = 0, units = 0;
    if (j < C) {
      const int c = brick_cell(j, n_c);
      int cnt = cell_count(start, c, n);
      if (cnt < occ_lo || cnt >= occ_hi) cnt = 0;   // only cells of this occupancy class
      if (active && cnt > 0) {   // only cells that hold an active slot
        const int a = min(max(start[c], 0), n);
        bool any = false;
        for (int k = a; k < a + cnt && !any; k += 8) {   // eight loads in flight
#pragma unroll
          for (int u = 0; u < 8; ++u) any |= active[min(k + u, a + cnt - 1)] != 0;
        }
        if (!any) cnt = 0;
      }
      if (merge > 1 && cnt > 0 && cnt <= ti) {
        const int m = merge_group(start, n, n_c, ti, merge, occ_lo, occ_hi, c);
        items = m > 0 ? 1 : 0;         // the group's first cell holds its one item
      } else {
        items = (cnt + ti - 1) / ti;
      }
      if (cnt > 0) {
        int cx, cy, cz;
        cell_coords(c, n_c, cx, cy, cz);
        int64_t nb = 0;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
          const int y = (cy + q % 3 - 1 + n_c) % n_c, z = (cz + q / 3 - 1 + n_c) % n_c;
          nb += row_count(start, n_c, n, n_c * (y + n_c * z), cx);
        }
        // a chunk stages about the particles within a support radius of it; with
        // h following the density that is a bounded number even next to crowded
        // cells, so the neighbour count is capped at that of a 64-per-cell lattice
        const int64_t raw = (int64_t)cnt * min(nb, (int64_t)kNbCap);
        const int64_t u = (raw + (1 << kCostShift) - 1) >> kCostShift;
        units = (int)min(u, (int64_t)cost_cap);
      }
    }
    uint64_t total;
    const uint64_t pre = carry + block_prefix(pair64(items, units), total, lds);
    carry += total;
    if (j < C && j != j0) {
      pos[j] = items_of(pre);
      cost[j] = cost_of(pre);
    }
  }
  if (threadIdx.x == 0) {
    pos[j0] = items_of(carry);
    cost[j0] = cost_of(carry);
  }
}

// Writes the items, and the range boundaries: range q starts at the first item
// of the first cell (in brick order) whose cost prefix reaches q/8 of the
// total, so the cell before it writes the boundary.
__global__ __launch_bounds__(kThreads) void k_wl_fill(const int32_t* __restrict__ start, int n_c,
                                                       int n, int ti, int capacity, int rounds,
                                                       int merge, int occ_lo, int occ_hi,
                                                       const int32_t* __restrict__ pos,
                                                       const int32_t* __restrict__ cost,
                                                       int2* __restrict__ items,
                                                       int32_t* __restrict__ counters,
                                                       int32_t* __restrict__ meta,
                                                       const int32_t* gate) {
  __shared__ uint64_t lds[kThreads / 64];
  if (gate && *gate == 0) return;
  const int C = n_c * n_c * n_c;
  const int span = rounds * kThreads, j0 = blockIdx.x * span;
  // totals of the blocks: those before this one, and all
  uint64_t before = 0, sum = 0;
#pragma unroll
  for (int i = 0; i < kMaxBlocks / kThreads; ++i) {
    const int b = i * kThreads + threadIdx.x;
    if (b < (int)gridDim.x) {
      const uint64_t v = pair64(pos[b * span], cost[b * span]);
      sum += v;
      before += b < (int)blockIdx.x ? v : 0;
    }
  }
  uint64_t base, all;
  block_prefix(before, base, lds);
  block_prefix(sum, all, lds);
  const int total = min(items_of(all), capacity);
  const int64_t cost_all = cost_of(all);
  if (blockIdx.x == 0 && threadIdx.x <= kQueues) {
    const int q = threadIdx.x;
    if (q == 0) meta[0] = total;
    if (q == 0 || q == kQueues || cost_all == 0) {
      meta[1 + q] = q == kQueues ? total : 0;
      if (q < kQueues) counters[q] = 0;
    }
  }
  for (int r = 0; r < rounds; ++r) {
    const int j = j0 + r * kThreads + threadIdx.x;   // position in brick order
    if (j >= C) return;
    const int je = min(j0 + span, C);
    const int lp = j == j0 ? 0 : pos[j], lc = j == j0 ? 0 : cost[j];
    const int np = j + 1 < je ? pos[j + 1] : pos[j0], nc = j + 1 < je ? cost[j + 1] : cost[j0];
    int o = items_of(base) + lp;
    const int next = items_of(base) + np;
    const int64_t c0 = (int64_t)cost_of(base) + lc, c1 = (int64_t)cost_of(base) + nc;
    if (c1 > c0) {
      for (int q = 1; q < kQueues; ++q) {
        const int64_t target = (cost_all * q + kQueues - 1) / kQueues;
        if (c0 < target && target <= c1) {
          meta[1 + q] = min(next, total);
          counters[q] = min(next, total);
        }
      }
    }
    const int end = min(next, capacity);   // this cell's items (none if filtered out)
    if (o >= end) continue;
    const int c = brick_cell(j, n_c);
    const int a = min(max(start[c], 0), n), b = min(max(start[c + 1], a), n);
    if (merge > 1 && b - a <= ti) {   // one item: the cell or its merged group
      const int m = max(merge_group(start, n, n_c, ti, merge, occ_lo, occ_hi, c), 1);
      items[o] = make_int2(c | ((m - 1) << kMergeShift), a);
      continue;
    }
    for (int f = a; f < b && o < end; f += ti, ++o) items[o] = make_int2(c, f);
  }
}

}  // namespace

int worklist_capacity(int n, int n_c, int ti) {
  const int64_t C = (int64_t)n_c * n_c * n_c;
  const int64_t t = ti > 0 ? ti : 1;
  const int64_t occupied = C < n ? C : n;
  const int64_t cap = (n + (t - 1) * occupied) / t + 1;
  return (int)(cap < (1LL << 30) ? cap : (1LL << 30));
}

size_t worklist_bytes(int n, int n_c, int ti) {
  const int C = n_c * n_c * n_c;
  const int cap = worklist_capacity(n, n_c, ti);
  return kWorkHeader + 2 * al256(sizeof(int32_t) * ((size_t)C + 1)) + sizeof(int2) * (size_t)cap;
}

hipError_t launch_worklist(const CellsDev& c, const WorkDev& w, hipStream_t s) {
  return launch_worklist_active(c, w, nullptr, s);
}

hipError_t launch_worklist_active(const CellsDev& c, const WorkDev& w, const uint8_t* active,
                                  hipStream_t s) {
  return launch_worklist_range(c, w, active, 0, 0x7fffffff, s);
}

hipError_t launch_worklist_range(const CellsDev& c, const WorkDev& w, const uint8_t* active,
                                 int occ_lo, int occ_hi, hipStream_t s, const int32_t* gate) {
  const int C = c.n_c * c.n_c * c.n_c;
  WlLayout L = wl_layout(reinterpret_cast<char*>(w.counters), C);
  const int cost_cap = (int)((((int64_t)1 << 31) - 1) / ((int64_t)C + 1));
  // merged items only for plain lists (the h iteration's lists filter cells)
  const int merge = active ? 1 : w.merge;
  const int rounds = wl_rounds(C), blocks = cdiv(C, rounds * kThreads);
  k_wl_count<<<blocks, kThreads, 0, s>>>(c.start, c.n_c, c.n, w.ti, cost_cap, rounds, active,
                                         occ_lo, occ_hi, merge, L.pos, L.cost, gate);
  k_wl_fill<<<blocks, kThreads, 0, s>>>(c.start, c.n_c, c.n, w.ti, w.capacity, rounds, merge,
                                        occ_lo, occ_hi, L.pos, L.cost, w.items, w.counters,
                                        w.meta, gate);
  return hipGetLastError();
}

WorkDev work_view(const sph_work& w, int n, int n_c) {
  WorkDev d;
  d.ti = w.ti;
  d.sched = w.sched;
  d.capacity = worklist_capacity(n, n_c, w.ti);
  d.merge = w.max_cells > 1 ? min(w.max_cells, kMaxMerge) : 1;
  char* base = static_cast<char*>(w.buf);
  d.counters = reinterpret_cast<int32_t*>(base);
  d.meta = reinterpret_cast<int32_t*>(base + 64);
  const int C = n_c * n_c * n_c;
  d.items = wl_layout(base, C).items;
  return d;
}

}  // namespace sph
