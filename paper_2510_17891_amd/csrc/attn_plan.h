// Host-side planning of the decode attention: how a context is cut into segments (shared with the kernels) and
// which rows of a batch can have their leading segments computed once for several rows.
//
// The G samples of one prompt (Section 2.3) hold the prompt's full pages in common.  Rows of such sequences that
// also have the same context length are cut into the same segments, and the segments that lie inside the common
// pages see the same keys and values: they are computed once per set of rows.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "chip.h"

#if defined(__HIPCC__)
#define RL_HOST_DEVICE __host__ __device__
#else
#define RL_HOST_DEVICE
#endif

namespace rl {

// Segments of a context of ctx keys: their number, and the first 32-key step of segment sgm (n_it = steps of the
// context, n_seg = its segments; sgm <= n_seg <= 256 and n_it < 2^16, so the product fits 32 bits).
RL_HOST_DEVICE inline int attn_num_segments(int ctx) { return 4 * ((ctx + 1023) / 1024); }
RL_HOST_DEVICE inline int attn_seg_begin(int sgm, int n_it, int n_seg) {
  return (int)(((unsigned)sgm * (unsigned)n_it) / (unsigned)n_seg);
}

// Segments up to which a row is finished by one block, and the segments of a block beyond.
// A compute unit draws 63 GB/s from memory whatever is in flight, so a step of four waves of a block takes 1.05 us, that of a
// wave alone 0.7: rows that leave compute units idle take blocks of four, two or one segment, as few as still make no more
// than a block per unit.  That costs the merge launch (4.7 us by itself, 3 of a layer, whose other launches overlap its start and end), which from
// 1025 keys (eight segments: half the steps per wave) always pays, and with four segments of bf16 pages from some 350 keys on.  One layer, us, before / with several blocks:
//   1 row:  1000 keys 93.2 / 88.3, 1500 97.6 / 89.3, 3900 102.5 / 90.3, 7000 (blocks of four / of one) 96.8 / 92.5
//   2 rows of 2000 104.1 / 92.0;  4 rows: 1000 98.1 / 93.3, 2000 106.7 / 95.1, fp8 pages 99.7 / 94.1
//   8 rows: 1000 99.6 / 95.8, 1500 104.0 / 97.9, 3000 118.1 / 105.3
// The line at 384: 1 row of 150 keys 85.9 / 86.6, 300 87.1 / 87.2, 450 88.3 / 87.9, 600 89.5 / 88.4; 8 rows of 150 91.4 / 92.0,
// 450 94.4 / 93.6; four segments of fp8 pages, 4 rows of 500 keys, 91.3 / 92.6.
// (Sets have blocks of their own beside the rows': there the rows' stay as they are.)
constexpr int kLdsSegs = 16;         // contexts up to 4096 can keep their segment partials in LDS
constexpr int kAttnWholeKeys = 384;  // contexts that one block finishes at least as fast as several
struct AttnSplit {
  int whole_segs, spb;
};
inline AttnSplit attn_split(int n_rows, int n_kv, bool kv_fp8, int max_ctx, bool sets, int segs_per_block) {
  AttnSplit r = {kLdsSegs, std::min(std::max(segs_per_block, 1), kLdsSegs)};
  const int pairs = n_rows * n_kv, n_seg = attn_num_segments(max_ctx);
  if (sets || pairs * (n_seg / 4) > kComputeUnits) return r;
  const bool ones = pairs * n_seg <= kComputeUnits;
  r.whole_segs = ones && !kv_fp8 && max_ctx > kAttnWholeKeys ? 0 : 4;
  if (ones) r.spb = 1;
  else if (pairs * (n_seg / 2) <= kComputeUnits) r.spb = std::min(r.spb, 2);
  return r;
}

// The context that stands for contexts of max_ctx keys in a captured launch: the end of its 1024 keys, which have the segments of every
// context in them, or the line between one block and several where that lies between (a batch in lock step meets it once).
inline int attn_capture_ctx(int n_rows, int n_kv, bool kv_fp8, int max_ctx, bool sets) {
  const int end = (max_ctx + 1023) / 1024 * 1024;
  const auto whole = [&](int ctx) { return attn_split(n_rows, n_kv, kv_fp8, ctx, sets, 1).whole_segs; };
  return whole(max_ctx) == whole(end) ? end : kAttnWholeKeys;
}

// Rows of equal context length whose leading pages are the same physical pages: their first n_segs segments are
// computed once for the set.  n_segs == 0: a pack of up to four (row, segment) pairs, pair w being rows[w] and
// rows[kAttnPackSegs + w] (unused pairs repeat the first).
constexpr int kAttnSetRows = 8, kAttnPackSegs = 4;
struct AttnShared {
  int32_t rows[kAttnSetRows];  // entries beyond n_rows repeat rows[0]
  int32_t n_rows;
  int32_t n_segs;
};

// Rows a set may hold: the matrix operand has 16 columns of (row, query head of the kv head) pairs, and the kernel
// for bf16 pages can run two such operands side by side (the one for fp8 pages has the registers for one).  Two
// operands halve the reads of the common keys once more but make the set's blocks the longest of the launch, which
// pays only when the launch is large and bound by memory traffic: from 1024 (row, kv head) pairs on, four row blocks
// per compute unit (measured: a loss at 64 rows, even at 96 to 128 rows, a gain from 128 rows with long prompts on).
// The choice changes no bit of any result.
inline int attn_rows_per_set(int group, bool kv_fp8, int n_rows, int n_kv) {
  const int one_operand = std::min(4, 16 / group);
  if (kv_fp8 || n_rows * n_kv < 1024) return one_operand;
  return std::min(kAttnSetRows, 32 / group);
}

// The longest context up to which the rows of a decode step do better each on its own (0: sharing always pays).  Sets make a merge launch
// necessary (3 us of a layer), which rows alone that one block finishes do without (attn_split: up to 4096 keys, up to 384 or 1024 where
// few rows take several blocks); and set blocks take two segments or more, where the blocks of few rows
// alone take as few as fill the compute units.  What sets save: bytes, as soon as the blocks of a compute unit share what it draws from memory,
// and blocks, which few rows alone have to share a unit with beyond.  One layer, us, shared / each on its own (8 kv heads, groups of 8):
//   2 rows: 3900 keys 94.1 / 93.3, 7000 96.9 / 95.6;  4 rows: 2000 95.2 / 94.0, 3900 97.3 / 97.4, 5000 97.7 / 99.6, 7900 105.4 / 105.0
//   8 rows: 1500 95.9 / 94.9, 3000 99.1 / 98.3, 3900 101.7 / 101.1, 5000 103.6 / 106.3, fp8 pages 3900 99.5 / 98.3
//   16 rows: 1300 98.6 / 97.9, 1750 100.1 / 99.9, 2040 101.1 / 105.3, fp8 pages 1900 99.5 / 99.0
//   32 rows: 1200 104.5 / 102.5, 1450 105.3 / 105.0, 36 layers of 1025 3891 / 3797
//   48 rows: 600 120.0 / 119.5, 1000 124.6 / 125.3;  64 rows: 600 127.9 / 122.9, 800 129.5 / 125.9, 1000 130.2 / 129.4
//   80 rows: 300 135.0 / 130.5, 700 142.6 / 138.3, 900 142.2 / 142.8;  104 rows: 500 152.5 / 151.9, 700 154.6 / 158.3
//   120 rows: 300 153.9 / 151.1, 500 157.8 / 156.8, 700 159.7 / 162.0
// From 1024 pairs on (wide sets, packs), attention and merge: 128 rows of 300 keys 25.7 / 26.1, 600 30.9 / 35.1.
// Rows alone read a prompt's pages once each, and only the L2 of a die makes that bearable: the kv head is the fastest grid index, so its rows
// meet on one die where the kv heads are a multiple of the eight dies.  Otherwise every die reads the pages (one layer, us, sets of four samples /
// alone: 2 kv heads, 128 rows of 1456 keys 127.5 / 135.4, 64 of 896 97.5 / 99.9; 1 kv head, 256 of 1456 152.6 / 158.4).  With 16 kv heads as with
// 8 (4 rows of 2000 keys 93.1 / 91.0).  One query head per kv head: the larger steps lose (88 rows of 720 keys 112.2 / 117.2, 120 of 464
// 120.5 / 124.1) and the smaller ones gain nothing (all of them together 1.001).
inline int attn_alone_up_to(int n_rows, int n_kv, int group) {
  if (n_kv % kDies != 0 || group == 1) return 0;
  const int pairs = n_rows * n_kv;
  if (pairs <= 128) return pairs <= 16 ? 8192 : pairs <= 64 ? 4096 : 1792;
  if (pairs <= 256) return 1500;
  if (pairs <= 512) return 900;
  return pairs <= 704 ? 768 : pairs < 1024 ? 512 : 0;
}

// Leading segments of a context of ctx keys that end inside the first shared_keys keys.
inline int attn_shared_segments(int ctx, int shared_keys) {
  const int n_it = (ctx + 31) >> 5, n_seg = attn_num_segments(ctx);
  int s = 0;
  while (s < n_seg && attn_seg_begin(s + 1, n_it, n_seg) * 32 <= shared_keys) ++s;
  return s;
}

struct AttnPlan {
  std::vector<int32_t> skip;     // per row: leading segments some set covers
  std::vector<AttnShared> sets;
  int max_shared_segs = 0;
  int packs = 0;            // entries at the end of `sets` that are packs
  bool all_packed = false;  // no row is left to a block of its own
};

// prefix_id[i] != 0 names the page-sharing family of row i (equal ids: the first prefix_blocks[i] pages are the
// same physical pages), pos[i] is the row's position.  rows_per_set <= kAttnSetRows.
inline void plan_shared_attention(int n, const int64_t* prefix_id, const int32_t* prefix_blocks, const int32_t* pos,
                                  int rows_per_set, AttnPlan* plan) {
  plan->skip.assign(n, 0);
  plan->sets.clear();
  plan->max_shared_segs = 0;
  std::vector<int> order;
  for (int i = 0; i < n; ++i)
    if (prefix_id[i] != 0) order.push_back(i);
  std::sort(order.begin(), order.end(), [&](int a, int b) {
    if (prefix_id[a] != prefix_id[b]) return prefix_id[a] < prefix_id[b];
    if (pos[a] != pos[b]) return pos[a] < pos[b];
    return a < b;
  });
  size_t i = 0;
  while (i < order.size()) {
    size_t e = i + 1;
    while (e < order.size() && prefix_id[order[e]] == prefix_id[order[i]] && pos[order[e]] == pos[order[i]]) ++e;
    const int first = order[i];
    const int shared_keys = std::min(prefix_blocks[first] * 16, pos[first]);  // a row's own key is never shared
    const int segs = attn_shared_segments(pos[first] + 1, shared_keys);
    if (segs > 0) {
      for (size_t b = i; b + 1 < e; b += rows_per_set) {  // a single left-over row computes everything itself
        AttnShared s;
        s.n_rows = (int)std::min<size_t>(rows_per_set, e - b);
        s.n_segs = segs;
        for (int k = 0; k < kAttnSetRows; ++k) s.rows[k] = order[b + (k < s.n_rows ? k : 0)];
        for (int k = 0; k < s.n_rows; ++k) plan->skip[order[b + k]] = segs;
        plan->sets.push_back(s);
        plan->max_shared_segs = std::max(plan->max_shared_segs, segs);
      }
    }
    i = e;
  }
}

// Rows of sets with one to three segments left behind the shared ones: a block of their own would keep as many of its
// four waves busy, and a large launch lasts as many rounds of blocks as there are rows.  These segments are packed
// four to a block instead, one per wave.  A packed row's skip is one more than its segments (no row block does
// anything for it, and the merge does not take it for a row that a set has finished).  Nothing is packed in launches
// that put less than `min_pairs` (row, kv head) pairs on the chip, where each row's wave has a compute unit to itself,
// or where the list would outgrow `max_entries`.  padded: empty packs (n_rows == 0) follow, as many as make the number
// of entries depend on the packed rows alone and not on how many segments they have left (a graph's launch shape).
inline void plan_packs(int n, const int32_t* pos, int n_kv, int group, int min_pairs, int max_entries, bool padded, AttnPlan* plan) {
  plan->packs = 0;
  plan->all_packed = false;
  if (plan->sets.empty() || n * n_kv < min_pairs || group * 4 > 16) return;  // the four rows' heads share one operand
  int units = 0, rows = 0;
  const auto left = [&](int r) { return plan->skip[r] ? attn_num_segments(pos[r] + 1) - plan->skip[r] : 0; };
  const auto packed = [&](int r) { return left(r) >= 1 && left(r) <= 3; };
  bool all = true;
  for (int r = 0; r < n; ++r) {
    if (!packed(r)) {
      all = false;
      continue;
    }
    units += left(r);
    rows += 1;
  }
  const int entries = ((padded ? 3 * rows : units) + 3) / 4;
  if (!units || (int)plan->sets.size() + entries > max_entries) return;
  AttnShared s = {};  // no rows, no shared segments
  for (int r = 0; r < n; ++r) {
    if (!packed(r)) continue;
    const int n_seg = attn_num_segments(pos[r] + 1);
    for (int sgm = plan->skip[r]; sgm < n_seg; ++sgm) {
      for (int k = s.n_rows; k < kAttnPackSegs; ++k) {
        s.rows[k] = s.n_rows ? s.rows[0] : r;
        s.rows[kAttnPackSegs + k] = s.n_rows ? s.rows[kAttnPackSegs] : sgm;
      }
      s.rows[s.n_rows] = r;
      s.rows[kAttnPackSegs + s.n_rows] = sgm;
      if (++s.n_rows == kAttnPackSegs) {
        plan->sets.push_back(s);
        s.n_rows = 0;
      }
    }
    plan->skip[r] = n_seg + 1;
  }
  if (s.n_rows) plan->sets.push_back(s);
  s.n_rows = 0;
  for (int e = (units + 3) / 4; e < entries; ++e) plan->sets.push_back(s);
  plan->packs = entries;
  plan->all_packed = all;
}

// Segments of a set block of a decode step: four, or two in steps of few rows with long prompts, where
//   - those make no more than a block per compute unit: one layer, us, four / two: 8 rows of 5000 shared keys 106.0 / 103.6, 16 of 2500
//     103.2 / 101.8, 24 of 1700 107.5 / 102.9, 32 of 1700 107.0 / 106.6, 32 with 1024 of 1924 shared 124.2 / 122.4;
//   - and with the rows' own blocks no more than the two per unit that fit: 48 rows of 1008 keys, eight samples a prompt, 99.0 / 102.1 (576
//     blocks), 24 rows of 16 kv heads 95.9 / 99.0 (at 512 blocks four query heads per kv head gain 1 to 4 %, two lose 2);
//   - and no row is left to itself: such a row's blocks last as long as the launch, and with the set blocks on all units none runs beside idle ones
//     (20 rows of 2000 keys, 16 of them in sets of four, 0.946 times as fast with two; two query groups of eight, 18 rows of 5008 keys
//     in sets of two and alone, 0.940; all such sizes together 0.966 to 1.010).
// Four / one: 16 rows with 1500 of 2500 shared keys 111.9 / 113.0; fp8 pages, 16 rows of 3000, four / two and less 99.6 / 102.6.
inline int attn_set_segments(int n_rows, int n_kv, bool kv_fp8, const AttnPlan& plan) {
  const int blocks = (int)plan.sets.size() * n_kv * ((plan.max_shared_segs + 1) / 2);
  const bool alone = std::find(plan.skip.begin(), plan.skip.end(), 0) != plan.skip.end();
  return kv_fp8 || plan.packs || alone || blocks > kComputeUnits || blocks + n_rows * n_kv > 2 * kComputeUnits ? 4 : 2;
}

// Rows that feed consecutive positions of one sequence (prefill, scoring).  Positions inside one aligned window of
// 32 have the same number of 32-key steps and hence the same segments, and every row's keys are a prefix of the
// keys of the row after it: up to rows_per_set (<= kAttnSetRows) neighbouring rows of a window form a set that computes ALL their
// segments side by side (n_segs = every segment, each column masked at its own context length), so the window's
// keys are read once per set instead of once per row.  rows[0] of a set is its highest position (the block takes
// its page list and step count from it).  seq[i], pos[i]: sequence and position of row i; rows of a sequence must
// be adjacent and ascending, as the chunks of a prefill are.
inline void plan_window_sets(int n, const int32_t* seq, const int32_t* pos, int rows_per_set, AttnPlan* plan) {
  plan->skip.assign(n, 0);
  plan->sets.clear();
  plan->max_shared_segs = 0;
  int i = 0;
  while (i < n) {
    int e = i + 1;
    while (e < n && e - i < rows_per_set && seq[e] == seq[i] && pos[e] == pos[e - 1] + 1 && (pos[e] >> 5) == (pos[i] >> 5)) ++e;
    if (e - i >= 2) {
      AttnShared s;
      s.n_rows = e - i;
      s.n_segs = attn_num_segments(pos[e - 1] + 1);  // the same for every member
      for (int k = 0; k < kAttnSetRows; ++k) s.rows[k] = e - 1 - (k < s.n_rows ? k : 0);
      for (int k = i; k < e; ++k) plan->skip[k] = s.n_segs;
      plan->sets.push_back(s);
      plan->max_shared_segs = std::max(plan->max_shared_segs, s.n_segs);
    }
    i = e;
  }
}

}  // namespace rl
