// How truncated sampling cuts the rows of a call (host and device; no GPU calls, unit-tested on the CPU): every row into
// slices, one block each, and a slice into units of 64 groups of four logits.
#pragma once

#include <algorithm>

#if defined(__HIPCC__)
#define RL_CUT_HD __host__ __device__
#else
#define RL_CUT_HD
#endif

namespace rl {

constexpr int kCutSlices = 32;  // at most, per row
constexpr int kCutTile = 2048;  // logits of a slice, at least
// Units of a row whose largest logit is kept: those of 2^18 logits, and one more per slice, which may end in the middle of one.
constexpr int kCutUnits = 1024 + kCutSlices;

// Slices per row of a call of M rows.  Two blocks per compute unit: every block clears, scans or flushes a histogram of its own.
// Three, which is what the LDS of the third pass allows, where there are logits enough for them.  Two -> three, us at 0.6 / 0.95
// and at 1.0 / 0.95: 128 rows of 151936 entries 61.3 -> 60.1 and 86.9 -> 83.2, 95 of 102400 (9.7 M logits) 45.9 -> 45.4 and 58.5
// -> 54.6, 64 of 151936 (9.7 M) 42.7 -> 42.9 and 53.7 -> 53.0, 72 of 128000 (9.2 M) no difference; but 64 of 128000 (8.2 M) 40.4
// -> 41.9 and 49.6 -> 49.8, 128 of 65536 (8.4 M) 42.2 -> 44.1 and 50.1 -> 51.9, 48 of 151936 (7.3 M) 39.2 -> 41.8 and 46.7 -> 48.3.
inline int cut_slices(int M, int V) {
  const int slices = ((long long)M * V >= 9000000 ? 768 : 512) / M;
  return std::max(1, std::min(std::min(slices, kCutSlices), (V + kCutTile - 1) / kCutTile));
}

RL_CUT_HD inline int cut_groups_per_slice(int V, int slices) { return ((V >> 2) + slices - 1) / slices; }
RL_CUT_HD inline int cut_units_per_slice(int V, int slices) { return (cut_groups_per_slice(V, slices) + 63) >> 6; }
// Whether the row keeps its units' largest logits.
RL_CUT_HD inline bool cut_keeps_units(int V, int slices) { return slices * cut_units_per_slice(V, slices) <= kCutUnits; }

}  // namespace rl
