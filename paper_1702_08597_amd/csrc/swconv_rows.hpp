// How a group of lanes walks a CSR row.  Plain C++, so that the arithmetic can be run on the host over the whole
// range of int32 row pointers.
#pragma once
#include <cstdint>

namespace swconv {

// Stored entries of row [q0, q1); a row that runs backwards has none.
constexpr uint32_t row_entries(int32_t q0, int32_t q1) { return q1 > q0 ? (uint32_t)q1 - (uint32_t)q0 : 0u; }

// f(i, n) for every chunk of kLanes entries of a row of n: lane l of the group works on entry i + l of the row while
// i + l < n, every lane of the group comes through every chunk.  Entries count from the row's start and unsigned: the
// position in the arrays, q0 + i + l, passes the int32 range in the last chunk of a row that ends near 2^31.
template <uint32_t kLanes, typename F>
constexpr void for_row_chunks(int32_t q0, int32_t q1, F&& f) {
  const uint32_t n = row_entries(q0, q1);
  for (uint32_t i = 0; i < n; i += kLanes) f(i, n);
}

// The two entry-wise kernels of the pruning step: 16 lanes to a row, kPruneRows rows per workgroup.
constexpr int kPruneRowLanes = 16;
constexpr int kPruneThreads = 256;
constexpr int kPruneRows = kPruneThreads / kPruneRowLanes;

// Up to here the second of them finds its row pointers itself, from one sum per workgroup of the first: a thread then
// reads at most kPruneLocalTurns of them.  (The sums that all workgroups read together grow with the square of the rows.
// Whole steps without and with a scan between the two, 3 and 25 entries a row, us: 13 824 rows 8.6, 10.0 and 12.8, 14.3;
// 24 576 12.3, 14.0 and 18.7, 20.9; 32 768 20.3, 23.3 and 19.7, 22.4; 49 152 36.3, 39.8 and 27.5, 31.7; 65 536 50.6, 55.8 and 34.5, 39.8.)
constexpr int kPruneLocalTurns = 8;
constexpr int64_t kPruneLocalRows = (int64_t)kPruneLocalTurns * kPruneThreads * kPruneRows;

// Their workgroups: one per kPruneRows rows up to 2^23; beyond 2^27 rows a workgroup takes more than one turn.  A launch
// of 2^32 threads or more wraps: rows were skipped without an error.  Any row count that int32 row pointers can number.
constexpr unsigned prune_groups(int64_t rows) {
  const int64_t groups = (rows + kPruneRows - 1) / kPruneRows, most = (int64_t)1 << 23;
  return (unsigned)(groups < most ? groups : most);
}

}  // namespace swconv
