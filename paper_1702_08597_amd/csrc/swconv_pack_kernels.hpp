// Packing of a sparse operand on the device: from per-position CSR arrays (or from the packed W_F, for its
// transpose) to the sliced layout of the sparse product, its slice descriptors and its schedule.
//
// A training loop that prunes changes the pattern in every step, so this is on its path.  On the host the
// same work (copy to the host, sort, fill, cut the schedule, copy back) took 2.6 ms for the forward operand
// of the 256 -> 384, N = 32, F(4x4,3x3) layer at 10 % density and 2.2 ms for its transpose; here the two take
// 50 us (9 + 10 us of kernels, the rest are the two waits for the host's part) and 25 us (13 + 11).  Everything is a
// gather or scatter of a few MB; what bounds it are chains of dependent loads and, in the sorts, that one workgroup per
// position leaves 64 of 256 CUs with work at most.
//   launch 1  one workgroup per position sorts the rows by length and takes the prefix sums over its slices
//             (forward: the column indices are validated by further workgroups of the same launch)
//   launch 2  slice descriptors and stream, one wave per slice; one more workgroup cuts the schedule
// The result does not depend on the order in which anything runs: ranks come from comparisons and bit
// counts, never from atomics, and equal the ranks of the host's stable sort.
#pragma once
#include "swconv_kernels.hpp"
#include "swconv_rows.hpp"

namespace swconv {

constexpr int kPackThreads = 1024;     // threads of a packing workgroup: 16 waves
constexpr int kPackMaxRows = 4096;     // rows per position that a packing workgroup sorts (its keys: 16 KB of LDS)
constexpr int kPackCheckRows = 128;    // rows per column-checking workgroup, 16 lanes to a row
constexpr int kPackMaxWgs = 1024;      // ranges that the schedule's workgroup cuts, one per thread
constexpr int kMaxPositions = 64;
constexpr int kCutStaged = 8192;       // prefix sums that the schedule's workgroup holds in LDS
constexpr int kFillBatches = 4;        // batches of a slice whose entries are on their way together
constexpr int kPackSpareWgs = 16;      // workgroups of launch 2 that clear the pairs behind the last slice

// What launch 1 says about a position.
struct PositionStats {
  int32_t batches;  // 512-byte stream batches of its slices
  int32_t cost;     // schedule cost of its slices: their lengths and slice_ovh for each
  int32_t longest;  // stored entries of its longest row
};

// Launch 1's tables of one operand, per position: rows in sorted order, and exclusive prefix sums over
// its slices (one more entry than slices, the last one is the total).
struct PackTables {
  int32_t* order;       // [P][rows_padded] original row of each sorted row, -1 = padding
  int32_t* len;         // [P][rows_padded] stored entries of each sorted row
  int32_t* batch_pre;   // [P][slices + 1]
  int32_t* cost_pre;    // [P][slices + 1]
  PositionStats* stats; // [P]
};

// ---- schedule ----

struct ScheduleShape {
  int P, ntb, spp;        // positions, tile blocks, slices per position
  int item_cap;           // most slices of a work item
  int n_launch;           // ranges = workgroups, at most the number of units
  int cus;                // compute units: the workgroups beyond them are second on their CU
  int second_share;       // percent of a first workgroup's budget that a second one gets
  int slice_ovh;          // cost of a slice besides its steps
  int panel_cost;         // cost of entering a panel
};

// Whether the workgroup that runs range r arrives second on its CU (ids are dealt one per CU first; the
// id follows from xcd_contiguous_id).
__host__ __device__ inline bool second_on_cu(int r, const ScheduleShape& s) {
  const int per = s.n_launch / kXcds, rem = s.n_launch % kXcds;
  const int head = rem * (per + 1);
  const int xcd = r < head ? r / (per + 1) : rem + (r - head) / (per > 0 ? per : 1);
  const int local = r - (xcd * per + (xcd < rem ? xcd : rem));
  return local * kXcds + xcd >= s.cus;
}

// Budgets: the ranges get shares of the work, 100 or second_share, and every range after the first is taken to
// pay one panel for starting inside one.  What is left of a range's budget after that is its net budget.
__device__ inline double range_share(int r, const ScheduleShape& s) {
  return second_on_cu(r, s) ? s.second_share : 100;
}
__device__ inline double net_budget(int r, double total, double shares, const ScheduleShape& s) {
  const double budget = range_share(r, s) * ((total + (double)(s.n_launch - 1) * s.panel_cost) / shares);
  const double net = budget - (r > 0 ? s.panel_cost : 0);
  return net < budget / 8 ? budget / 8 : net;
}
// First unit (of the sequence (position, tile block, slice)) at or after cumulative cost `target`.
// block_cost[p] = cost of all panels of the positions before p; pre(i) = entry i of cost_pre.
// (Moving cuts that fall near a panel boundary onto it saves a few panels and costs more in balance: the
// heaviest range of the 256 -> 384, N = 32 layer then has 7052 units instead of 6183.)
template <typename Pre>
__device__ inline int locate_unit(double target, const double* block_cost, Pre&& pre, const ScheduleShape& s) {
  int p = 0, end = s.P;  // the last position that begins at or before the target (the costs before them rise)
  while (p + 1 < end) {
    const int mid = (p + end) / 2;
    if (block_cost[mid] <= target) p = mid; else end = mid;
  }
  const int c = p * (s.spp + 1);
  const double a = (double)s.panel_cost + pre(c + s.spp);
  const double rem = target - block_cost[p];
  int tb = (int)(rem / a);
  tb = tb < 0 ? 0 : tb >= s.ntb ? s.ntb - 1 : tb;
  const double off = rem - tb * a;
  const int unit0 = (p * s.ntb + tb) * s.spp;
  int lo = 0, hi = s.spp;  // the last slice boundary at or before the target
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (pre(c + mid) + s.panel_cost <= off) lo = mid; else hi = mid - 1;
  }
  // the nearer of the two boundaries around it
  if (lo < s.spp && 2 * (off - s.panel_cost) > (double)pre(c + lo) + pre(c + lo + 1)) ++lo;
  return unit0 + lo;
}

// Work items of units [u0, u1): one per panel touched, none with more than item_cap slices.
template <typename F>
__device__ inline int for_items(int u0, int u1, const ScheduleShape& s, F&& emit) {
  int n = 0;
  while (u0 < u1) {
    const int pt = u0 / s.spp, s0 = u0 - pt * s.spp;
    int cnt = u1 - u0;
    cnt = cnt < s.spp - s0 ? cnt : s.spp - s0;
    cnt = cnt < s.item_cap ? cnt : s.item_cap;
    const int p = pt / s.ntb;
    emit(n, WorkItem{p, pt - p * s.ntb, p * s.spp + s0, p * s.spp + s0 + cnt});
    ++n;
    u0 += cnt;
  }
  return n;
}

// ---- device helpers ----

// Exclusive scan of one value per thread over a workgroup of kPackThreads; *total = the sum.  `part`: 17 words.
template <typename T>
__device__ __forceinline__ T block_scan(T x, T* part, T* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T incl = x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const T up = __shfl_up(incl, d);
    if (lane >= d) incl += up;
  }
  __syncthreads();  // the caller may still read `part` of a scan before
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  T before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kPackThreads / 64; ++w) {
    const T v = part[w];
    if (w < wave) before += v;
    all += v;
  }
  *total = all;
  return before + incl - x;
}

// Sorts one position's rows by length, longest first, equal ones in their order, and takes the prefix sums
// over its slices.  key[i] = (length + 1) << 12 | (4095 - i), zero from `rows` to the next multiple of four: a
// row's rank is the number of larger keys, counted by reading all keys as broadcasts, four at a time (signs of
// differences: keys are below 2^31).  Where the workgroup has threads for every row several times over, each
// counts a part of the keys and the parts are added in LDS (whole numbers: in any order).
// lds: 3 * rows_padded words on a 16-byte boundary, the keys first; the sorted keys are left in the second part.  (Off the
// boundary - the array behind 68 static bytes - a 16-byte read takes 64 clocks instead of four: 15 of
// pack_sort_kernel's 20.5 us at 384 rows.)
__device__ inline uint32_t* sort_position(int p, int rows, int rows_padded, uint32_t* lds, const PackTables& t, int slice_ovh) {
  __shared__ int32_t part[17];
  const uint32_t* key = lds;
  uint32_t* sorted = lds + rows_padded;
  int32_t* rank = reinterpret_cast<int32_t*>(lds) + 2 * rows_padded;
  const int spp = rows_padded / kSliceRows;
  for (int i = threadIdx.x; i < rows_padded; i += kPackThreads) {
    sorted[i] = 0u;
    rank[i] = 0;
  }
  __syncthreads();
  const int lanes = (rows + 63) / 64 * 64, quads = (rows + 3) / 4;  // a wave works on one part of the keys
  const int parts = max(1, min(kPackThreads / lanes, 8)), per_part = (quads + parts - 1) / parts;
  for (int i = threadIdx.x; i < lanes * parts; i += kPackThreads) {
    const int row = i % lanes, first = i / lanes * per_part, last = min(quads, first + per_part);
    if (row >= rows) continue;
    const uint32_t mine = key[row];
    int larger = 0;
#pragma unroll 8
    for (int j = first; j < last; ++j) {
      const uint4 k = *reinterpret_cast<const uint4*>(key + 4 * j);
      larger += (int)((mine - k.x) >> 31) + (int)((mine - k.y) >> 31) + (int)((mine - k.z) >> 31) + (int)((mine - k.w) >> 31);
    }
    atomicAdd(&rank[row], larger);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < rows; i += kPackThreads) sorted[rank[i]] = key[i];
  __syncthreads();
  auto length = [&](uint32_t k) { return k == 0u ? 0 : (int)(k >> 12) - 1; };
  for (int i = threadIdx.x; i < rows_padded; i += kPackThreads) {
    const uint32_t k = sorted[i];
    t.order[(size_t)p * rows_padded + i] = k == 0u ? -1 : 4095 - (int)(k & 4095u);
    t.len[(size_t)p * rows_padded + i] = length(k);
  }
  const int s = threadIdx.x;  // kPackMaxRows / kSliceRows slices at most: one per thread
  int steps = 0;
  if (s < spp) steps = (length(sorted[s * kSliceRows]) + kStepGroup - 1) / kStepGroup * kStepGroup;
  const int batches = (steps + kBatchSteps - 1) / kBatchSteps;
  int all_batches, all_cost;
  const int b0 = block_scan(batches, part, &all_batches);
  const int c0 = block_scan(s < spp ? steps + slice_ovh : 0, part, &all_cost);
  if (s < spp) {
    t.batch_pre[(size_t)p * (spp + 1) + s] = b0;
    t.cost_pre[(size_t)p * (spp + 1) + s] = c0;
  }
  if (s == 0) {
    t.batch_pre[(size_t)p * (spp + 1) + spp] = all_batches;
    t.cost_pre[(size_t)p * (spp + 1) + spp] = all_cost;
    t.stats[p] = PositionStats{all_batches, all_cost, length(sorted[0])};
  }
  return sorted;
}

// What the host reads of the packing of a forward operand (pinned host memory).
struct PackReport {
  // after launch 1
  int32_t nnz;
  int32_t bad;  // rowptr[0] != 0
  PositionStats stats[kMaxPositions];
  int32_t bad_rows[kMaxPositions];  // a row of the position leaves [0, nnz], is too long or runs backwards
  // after launch 2, of the schedule
  int32_t items;
  uint32_t heaviest_steps;  // slice steps of the workgroup with the most of them
};

// Launch 1 of a forward operand.  Grid (P, 1 + ceil(K / kPackCheckRows)): workgroup (p, 0) sorts position p,
// workgroup (p, j) checks the column indices of its rows and writes bad_cols[p * (gridDim.y - 1) + j - 1].
// No column of a row is read unless the row lies inside [0, nnz] with nnz <= P*K*C.
__global__ __launch_bounds__(kPackThreads) void pack_sort_kernel(const int32_t* __restrict__ rowptr,
                                                                 const int32_t* __restrict__ colidx, int P, int K,
                                                                 int rows_padded, int C, PackTables t, int slice_ovh,
                                                                 PackReport* __restrict__ report,
                                                                 int32_t* __restrict__ bad_cols) {
  extern __shared__ __attribute__((aligned(16))) uint32_t pack_lds[];
  const int p = blockIdx.x;
  const int32_t* rp = rowptr + (size_t)p * K;
  const int32_t nnz = rowptr[(size_t)P * K];
  const bool nnz_ok = nnz >= 0 && (int64_t)nnz <= (int64_t)P * K * C;
  auto row_ok = [&](int32_t a, int32_t b) { return nnz_ok && a >= 0 && a <= b && b <= nnz && b - a <= C; };
  if (blockIdx.y == 0) {
    uint32_t* key = pack_lds;
    int bad = 0;
    for (int i = threadIdx.x; i < rows_padded; i += kPackThreads) {
      uint32_t k = 0u;
      if (i < K) {
        const int32_t a = rp[i], b = rp[i + 1];
        const bool ok = row_ok(a, b);
        bad |= !ok;
        k = (uint32_t)((ok ? b - a : 0) + 1) << 12 | (uint32_t)(4095 - i);
      }
      key[i] = k;
    }
    bad = __syncthreads_or(bad);
    sort_position(p, K, rows_padded, key, t, slice_ovh);
    __syncthreads();
    if (threadIdx.x == 0) {
      report->stats[p] = t.stats[p];
      report->bad_rows[p] = bad;
      if (p == 0) {
        report->nnz = nnz;
        report->bad = rowptr[0] != 0;
      }
    }
    return;
  }
  int bad = 0;
  const int k_end = min(K, (int)blockIdx.y * kPackCheckRows);
  for (int k = ((int)blockIdx.y - 1) * kPackCheckRows + (int)(threadIdx.x >> 4); k < k_end; k += kPackThreads / 16) {
    const int32_t a = rp[k], b = rp[k + 1];
    if (colidx == nullptr || !row_ok(a, b)) continue;  // the host rejects a missing array by nnz alone
    for_row_chunks<16>(a, b, [&](uint32_t i, uint32_t n) {
      const uint32_t e = i + (threadIdx.x & 15);
      if (e >= n) return;
      const size_t q = (size_t)a + e;
      const int32_t c = colidx[q], before = e > 0 ? colidx[q - 1] : -1;
      bad |= c <= before || c >= C;
    });
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) bad_cols[p * ((int)gridDim.y - 1) + (int)blockIdx.y - 1] = bad;
}

// First batch of position p in the stream: the batches of the positions before it.
__device__ __forceinline__ int position_batch0(const PositionStats* stats, int p) {
  int n = (int)(threadIdx.x & 63) < p ? stats[threadIdx.x & 63].batches : 0;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) n += __shfl_xor(n, d);
  return n;
}

// The schedule: one workgroup, one range per thread.  The net budgets, scaled to the whole work, say where the
// ranges begin; the cuts are located in the prefix sums, made strictly ascending - no range is empty - and
// written as work items.  `report` (or null) gets the schedule's two statistics.
__device__ inline void cut_schedule(const ScheduleShape& s, const PackTables& t, WorkItem* items, RangeHeader* ranges,
                                    PackReport* report) {
  __shared__ double block_cost[kMaxPositions + 1];
  __shared__ uint32_t work_before[kMaxPositions];  // the same without the panels, modulo 2^32
  __shared__ uint32_t steps_at[kPackMaxWgs + 1];   // slice steps in front of a cut, modulo 2^32
  __shared__ uint32_t heaviest;
  __shared__ int32_t cut[kPackMaxWgs + 1];
  __shared__ double dpart[17];
  __shared__ int32_t ipart[17];
  // The searches below are chains of dependent reads, of memory for 1.5 us and more: the prefix sums come to LDS where
  // they fit (256 -> 384 channels: 3492 of them; 11.8 -> 9.8 us for the kernel, whose longest workgroup this is).
  __shared__ int32_t staged[kCutStaged];
  const int r = threadIdx.x, n_pre = s.P * (s.spp + 1);
  const bool stage = n_pre <= kCutStaged;
  if (stage)
    for (int i = r; i < n_pre; i += kPackThreads) staged[i] = t.cost_pre[i];
  auto pre = [&](int i) -> int32_t { return stage ? staged[i] : t.cost_pre[i]; };
  if (r < 64) {  // one position per lane (kMaxPositions); the sums are of whole numbers, so their order does not matter
    const int32_t cost = r < s.P ? t.stats[r].cost : 0;
    const double own = r < s.P ? (double)s.ntb * ((double)s.panel_cost + cost) : 0;
    const uint32_t own_work = (uint32_t)s.ntb * (uint32_t)cost;
    double sum = own;
    uint32_t work = own_work;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const double up = __shfl_up(sum, d);
      const uint32_t up_work = (uint32_t)__shfl_up((int)work, d);
      if (r >= d) sum += up, work += up_work;
    }
    if (r < s.P) {
      block_cost[r] = sum - own;
      work_before[r] = work - own_work;
    }
    if (r == s.P - 1) {
      block_cost[s.P] = sum;
      steps_at[s.n_launch] = work - (uint32_t)s.slice_ovh * (uint32_t)(s.P * s.ntb * s.spp);
      heaviest = 0;
    }
  }
  __syncthreads();
  const double total = block_cost[s.P];
  const int n = s.n_launch;
  const double share = r < n ? range_share(r, s) : 0;
  double shares, net_total;
  (void)block_scan(share, dpart, &shares);
  const double net = r < n ? net_budget(r, total, shares, s) : 0;
  double at = block_scan(net, dpart, &net_total);
  at *= total / net_total;
  const int units = s.P * s.ntb * s.spp;
  int u = units;
  if (r < n) u = r == 0 ? 0 : locate_unit(at, block_cost, pre, s);
  // strictly ascending: u[r] - r must not fall (running maximum), nor pass units - n
  int v = r < n ? u - r : 0;
  {
    const int lane = r & 63, wave = r >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(v, d);
      if (lane >= d) v = max(v, up);
    }
    __syncthreads();
    if (lane == 63) ipart[wave] = v;
    __syncthreads();
    for (int w = 0; w < wave; ++w) v = max(v, ipart[w]);
  }
  v = min(v, units - n) + r;
  __syncthreads();
  if (r < n) {
    cut[r] = v;
    if (report != nullptr) {
      // a range holds less than 2^32 steps (V and M have 32-bit sizes), so differences may wrap on the way
      const int pt = v / s.spp, p = pt / s.ntb;
      const int c = p * (s.spp + 1);
      steps_at[r] = work_before[p] + (uint32_t)(pt - p * s.ntb) * (uint32_t)pre(c + s.spp) + (uint32_t)pre(c + v - pt * s.spp) -
                    (uint32_t)s.slice_ovh * (uint32_t)v;
    }
  }
  if (r == 0) cut[n] = units;
  __syncthreads();
  int count = 0;
  if (r < n) count = for_items(cut[r], cut[r + 1], s, [](int, const WorkItem&) {});
  if (report != nullptr) {
    uint32_t steps = r < n ? steps_at[r + 1] - steps_at[r] : 0u;
    for (int d = 32; d > 0; d >>= 1) steps = max(steps, (uint32_t)__shfl_xor((int)steps, d));
    if ((r & 63) == 0) atomicMax(&heaviest, steps);
  }
  int all;
  const int first = block_scan(count, ipart, &all);  // its barriers also stand between the maximum and its reader
  if (r == 0 && report != nullptr) {  // now, not at the end: the way to the host's memory overlaps with the items
    report->items = all;
    report->heaviest_steps = heaviest;
  }
  if (r < n) {
    RangeHeader h{};
    h.item_begin = first;
    h.item_end = first + count;
    for_items(cut[r], cut[r + 1], s, [&](int i, const WorkItem& w) {
      items[first + i] = w;
      if (i == 0) h.first = w;
      if (i <= 1) h.second_slice = w.slice_begin;
    });
    ranges[r] = h;
  }
}

// Where launch 2 writes an operand.
struct PackedOut {
  uint32_t* stream;  // pairs
  int32_t* index;    // per pair: its index in the caller's CSR arrays, -1 = padding
  Slice* slices;
  WorkItem* items;
  RangeHeader* ranges;
  uint32_t n_pairs;  // pairs the stream holds, spare ones included
};

// The descriptor of slice s of position p, and its padding rows' and padding steps' pairs;
// `load(row, e, u)` and then `store(pair, u)` are called for every stored entry, up to kFillBatches of them (u) loaded
// before the first is stored.  One wave, lane (q, i) on step 16 b + i of row q.
template <typename Load, typename Store>
__device__ __forceinline__ void fill_slice(int p, int s, int rows_padded, int batch0, const PackTables& t,
                                           const PackedOut& out, Load&& load, Store&& store) {
  const int spp = rows_padded / kSliceRows, lane = threadIdx.x & 63, q = lane >> 4;
  const int row = p * rows_padded + s * kSliceRows;
  const int my_row = t.order[row + q], my_len = t.len[row + q];
  batch0 += t.batch_pre[(size_t)p * (spp + 1) + s];
  const int longest = __shfl(my_len, 0);
  const int steps = (longest + kStepGroup - 1) / kStepGroup * kStepGroup;
  Slice sl;
  sl.batch0 = (uint32_t)batch0;
  sl.len = steps;
  sl.row0 = row;
  sl.p = p;
#pragma unroll
  for (int i = 0; i < kSliceRows; ++i) sl.k[i] = __shfl(my_row, 16 * i);
  if (lane == 0) out.slices[(size_t)p * spp + s] = sl;
  for (int b = 0; b * kBatchSteps < steps; b += kFillBatches) {
#pragma unroll
    for (int u = 0; u < kFillBatches; ++u) {
      const int e = (b + u) * kBatchSteps + (lane & 15);
      if (e < my_len) load(my_row, e, u);
    }
#pragma unroll
    for (int u = 0; u < kFillBatches; ++u) {
      const int e = (b + u) * kBatchSteps + (lane & 15);
      const uint32_t pair = (uint32_t)(batch0 + b + u) * 64u + (uint32_t)lane;
      if (e < my_len)
        store(pair, u);
      else if ((b + u) * kBatchSteps < steps) {
        *reinterpret_cast<uint2*>(out.stream + 2 * (size_t)pair) = make_uint2(0u, 0u);
        out.index[pair] = -1;
      }
    }
  }
}

// Pairs behind the last slice, up to the size the buffers were given (the value update and the weight gradient's sums
// walk them all), one of kPackSpareWgs workgroups' share of them.
__device__ __forceinline__ void fill_spare(const PackTables& t, int P, const PackedOut& out, int part) {
  const uint32_t used = (uint32_t)(position_batch0(t.stats, P - 1) + t.stats[P - 1].batches) * 64u;
  for (uint32_t pair = used + part * kPackThreads + threadIdx.x; pair < out.n_pairs; pair += kPackSpareWgs * kPackThreads) {
    *reinterpret_cast<uint2*>(out.stream + 2 * (size_t)pair) = make_uint2(0u, 0u);
    out.index[pair] = -1;
  }
}

// Launch 2 of a forward operand.  Grid 1 + kPackSpareWgs + P * ceil(slices / 16): the schedule, the spare
// pairs, then 16 slices per workgroup.
__global__ __launch_bounds__(kPackThreads) void pack_fill_kernel(const int32_t* __restrict__ rowptr,
                                                                 const int32_t* __restrict__ colidx,
                                                                 const float* __restrict__ vals, int K, int rows_padded,
                                                                 PackTables t, PackedOut out, ScheduleShape shape,
                                                                 PackReport* __restrict__ report) {
  if (blockIdx.x == 0) {
    if (shape.n_launch > 0) cut_schedule(shape, t, out.items, out.ranges, report);
    return;
  }
  if (blockIdx.x <= kPackSpareWgs) return fill_spare(t, shape.P, out, (int)blockIdx.x - 1);
  const int wg = (int)blockIdx.x - 1 - kPackSpareWgs;
  const int chunks = (shape.spp + 15) / 16;
  const int p = wg / chunks, s = wg % chunks * 16 + (int)(threadIdx.x >> 6);
  const int batch0 = position_batch0(t.stats, p);
  if (s >= shape.spp) return;
  const int32_t* rp = rowptr + (size_t)p * K;
  int32_t at[kFillBatches], col[kFillBatches];
  float val[kFillBatches];
  fill_slice(
      p, s, rows_padded, batch0, t, out,
      [&](int row, int e, int u) {
        at[u] = rp[row] + e;
        col[u] = colidx[at[u]];
        val[u] = vals[at[u]];
      },
      [&](uint32_t pair, int u) {
        *reinterpret_cast<uint2*>(out.stream + 2 * (size_t)pair) =
            make_uint2((uint32_t)col[u] * (uint32_t)(kTileBlock * sizeof(float)), __float_as_uint(val[u]));
        out.index[pair] = at[u];
      });
}

// ---- the transpose of the packed W_F, for the backward pass ----

// Launch 1.  One workgroup per position: the position's pattern as a bit matrix [C][words of K], whose row
// counts are the transposed rows' lengths; the matrix goes to memory with the exclusive bit count in front of
// every word, so that launch 2 finds the place of an entry (k, c) in the transposed row c - its k ascending -
// with one load and one bit count.
__global__ __launch_bounds__(kPackThreads) void transpose_sort_kernel(const uint32_t* __restrict__ stream,
                                                                      const int32_t* __restrict__ index,
                                                                      const Slice* __restrict__ slices, int spp, int K,
                                                                      int C, int rows_padded, int words, PackTables t,
                                                                      int slice_ovh, uint2* __restrict__ bits,
                                                                      int32_t* __restrict__ rank_of) {
  extern __shared__ __attribute__((aligned(16))) uint32_t pack_lds[];
  uint32_t *map = pack_lds, *key = pack_lds + (C * words + 3) / 4 * 4;
  const int p = blockIdx.x, lane = threadIdx.x & 63;
  for (int i = threadIdx.x; i < C * words; i += kPackThreads) map[i] = 0u;
  __syncthreads();
  // four slices of a wave at a time, the loads of a batch of each in flight together (one slice after
  // the other, a chain of a descriptor and, a batch, an index and an offset: 23.5 us for the kernel, so 18.5; 12.8 with
  // the keys on their boundary)
  constexpr int U = 4, W = kPackThreads / 64;
  for (int s0 = threadIdx.x >> 6; s0 < spp; s0 += U * W) {
    int k[U], len[U], longest = 0;
    size_t pair[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const Slice sl = slices[(size_t)p * spp + min(s0 + u * W, spp - 1)];
      const int q = lane >> 4;
      k[u] = q == 0 ? sl.k[0] : q == 1 ? sl.k[1] : q == 2 ? sl.k[2] : sl.k[3];
      len[u] = s0 + u * W < spp ? sl.len : 0;
      pair[u] = (size_t)sl.batch0 * 64 + lane;
      longest = max(longest, len[u]);
    }
    for (int e = 0; e < longest; e += kBatchSteps) {
      int32_t at[U];
      uint32_t offset[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        at[u] = -1;
        if (e < len[u]) at[u] = index[pair[u]], offset[u] = stream[2 * pair[u]];
        pair[u] += 64;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (at[u] >= 0)
          atomicOr(&map[(int)(offset[u] / (uint32_t)(kTileBlock * sizeof(float))) * words + (k[u] >> 5)], 1u << (k[u] & 31));
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < rows_padded; c += kPackThreads) {
    uint32_t before = 0;
    if (c < C)
      for (int w = 0; w < words; ++w) {
        const uint32_t m = map[c * words + w];
        bits[((size_t)p * C + c) * words + w] = make_uint2(m, before);
        before += __popc(m);
      }
    key[c] = c < C ? (before + 1) << 12 | (uint32_t)(4095 - c) : 0u;
  }
  __syncthreads();
  const uint32_t* sorted = sort_position(p, C, rows_padded, key, t, slice_ovh);
  __syncthreads();
  for (int i = threadIdx.x; i < C; i += kPackThreads) rank_of[(size_t)p * C + (4095 - (int)(sorted[i] & 4095u))] = i;
}

// Launch 2.  Grid 1 + kPackSpareWgs + P * chunks: the schedule, the spare pairs; workgroup (p, j) writes descriptors and
// padding of 16 slices of the transpose and moves the entries of 16 slices of W_F to their places.
__global__ __launch_bounds__(kPackThreads) void transpose_fill_kernel(const uint32_t* __restrict__ stream,
                                                                      const int32_t* __restrict__ index,
                                                                      const Slice* __restrict__ slices, int fw_spp, int C,
                                                                      int rows_padded, int words, int chunks,
                                                                      const uint2* __restrict__ bits,
                                                                      const int32_t* __restrict__ rank_of, PackTables t,
                                                                      PackedOut out, ScheduleShape shape) {
  if (blockIdx.x == 0) {
    if (shape.n_launch > 0) cut_schedule(shape, t, out.items, out.ranges, nullptr);
    return;
  }
  if (blockIdx.x <= kPackSpareWgs) return fill_spare(t, shape.P, out, (int)blockIdx.x - 1);
  const int wg = (int)blockIdx.x - 1 - kPackSpareWgs;
  const int p = wg / chunks, s = wg % chunks * 16 + (int)(threadIdx.x >> 6);
  const int batch0 = position_batch0(t.stats, p), lane = threadIdx.x & 63;
  if (s < shape.spp) fill_slice(p, s, rows_padded, batch0, t, out, [](int, int, int) {}, [](uint32_t, int) {});
  if (s >= fw_spp) return;
  const Slice sl = slices[(size_t)p * fw_spp + s];
  const int q = lane >> 4, k = q == 0 ? sl.k[0] : q == 1 ? sl.k[1] : q == 2 ? sl.k[2] : sl.k[3];
  // the loads of kFillBatches batches in flight together: the way of an entry is a chain of three loads
  for (int b0 = 0; b0 * kBatchSteps < sl.len; b0 += kFillBatches) {
    int32_t at[kFillBatches];
    uint2 pair[kFillBatches];
#pragma unroll
    for (int u = 0; u < kFillBatches; ++u) {
      at[u] = -1;
      if ((b0 + u) * kBatchSteps < sl.len) {
        const size_t from = ((size_t)sl.batch0 + b0 + u) * 64 + lane;
        at[u] = index[from];
        pair[u] = *reinterpret_cast<const uint2*>(stream + 2 * from);
      }
    }
    uint2 m[kFillBatches];
    int slot[kFillBatches];
#pragma unroll
    for (int u = 0; u < kFillBatches; ++u)
      if (at[u] >= 0) {
        const int c = (int)(pair[u].x / (uint32_t)(kTileBlock * sizeof(float)));
        m[u] = bits[((size_t)p * C + c) * words + (k >> 5)];
        slot[u] = rank_of[(size_t)p * C + c];
      }
    int32_t pre[kFillBatches];
#pragma unroll
    for (int u = 0; u < kFillBatches; ++u)
      if (at[u] >= 0) pre[u] = t.batch_pre[(size_t)p * (shape.spp + 1) + slot[u] / kSliceRows];
#pragma unroll
    for (int u = 0; u < kFillBatches; ++u)
      if (at[u] >= 0) {
        const int e = (int)m[u].y + __popc(m[u].x & ((1u << (k & 31)) - 1u));  // entries of row c before k
        const uint32_t first = (uint32_t)(batch0 + pre[u]);
        const size_t to =
            ((size_t)first + e / kBatchSteps) * 64 + (size_t)(slot[u] % kSliceRows) * kBatchSteps + e % kBatchSteps;
        *reinterpret_cast<uint2*>(out.stream + 2 * to) = make_uint2((uint32_t)k * (uint32_t)(kTileBlock * sizeof(float)), pair[u].y);
        out.index[to] = at[u];
      }
  }
}

// ---- W_F in the package format of the fused product + output transform kernels ----

// One wave per (position, chunk of 64 rows, slice): rows in their natural order, B batches per slice.
__global__ __launch_bounds__(kPackThreads) void pack_fused_kernel(const int32_t* __restrict__ rowptr,
                                                                  const int32_t* __restrict__ colidx,
                                                                  const float* __restrict__ vals, int K, int KC, int B,
                                                                  uint32_t* __restrict__ wpk, int32_t* __restrict__ index,
                                                                  uint8_t* __restrict__ lens) {
  constexpr int NW = kPackThreads / 64;
  const int p = blockIdx.x / KC, kc = blockIdx.x % KC, w = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane >> 4;
  const int k = (kc * NW + w) * kSliceRows + q;
  const int32_t q0 = k < K ? rowptr[(size_t)p * K + k] : 0, len = k < K ? rowptr[(size_t)p * K + k + 1] - q0 : 0;
  int longest = len;
  longest = max(longest, __shfl_xor(longest, 16));
  longest = max(longest, __shfl_xor(longest, 32));
  if (lane == 0)
    lens[((size_t)p * KC + kc) * NW + w] = (uint8_t)((longest + kStepGroup - 1) / kStepGroup * kStepGroup);
  for (int b = 0; b < B; ++b) {
    const int e = b * kBatchSteps + (lane & 15);
    const size_t pair = ((((size_t)p * KC + kc) * B + b) * NW + w) * 64 + lane;
    uint2 v = make_uint2(0u, 0u);
    if (e < len)
      v = make_uint2((uint32_t)colidx[q0 + e] * (uint32_t)(kTileBlock * sizeof(float)), __float_as_uint(vals[q0 + e]));
    *reinterpret_cast<uint2*>(wpk + 2 * pair) = v;
    index[pair] = e < len ? q0 + e : -1;
  }
}

}  // namespace swconv
