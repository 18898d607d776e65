// How the bf16 projections are cut into K splits, tiles and blocks (host only; no GPU calls, unit-tested on the CPU).
#pragma once

#include "chip.h"

namespace rl {

enum Epilogue : int { kEpiPartial = 0, kEpiSwiGLU = 1, kEpiSample = 2, kEpiResidual = 3 };

struct GemmPlan {
  int splits;       // K splits across blocks
  int kb_per_wave;  // 64-wide k blocks per wave
};

inline GemmPlan gemm_plan(int N, int K, int epi, bool allow_split) {
  const int KB = K >> 6;
  const int tiles = epi == kEpiSwiGLU ? (N >> 5) : (N >> 6);
  int S = 1;
  // Split K across blocks until about one block per CU exists; each wave keeps >= 2 k blocks.
  while (tiles * S < 256 && (KB % (S * 2 * 4) == 0) && KB / (S * 2 * 4) >= 2 && epi == kEpiPartial && allow_split) S *= 2;
  return GemmPlan{S, KB / (S * 4)};
}

// Tiles of two sizes (see gemm_bf16_mixed_kernel): used when the matrix has exactly three (row block, K split) units
// per compute unit.
inline bool gemm_mixed_fits(int N, int K, int epi, bool allow_split) {
  if (epi == kEpiSample) return false;
  const GemmPlan p = gemm_plan(N, K, epi, allow_split);
  const int row_blocks = (epi == kEpiSwiGLU ? 2 * N : N) >> 5;
  return row_blocks % 3 == 0 && row_blocks * p.splits == 3 * kComputeUnits;
}

// Blocks of the 128-row tiling for (N, K): it is used where they still fill the chip.
inline int gemm_wide_blocks(int N, int K, int epi, bool allow_split) {
  const GemmPlan p = gemm_plan(N, K, epi, allow_split);
  const int tiles = epi == kEpiSwiGLU ? (N >> 5) : (N >> 6);
  return ((tiles + 1) / 2) * (epi == kEpiPartial ? p.splits : 1);
}

// Whether an M x N x K product of more than 256 rows runs over the whole K range in one block (gemm_bf16_tile_kernel with
// running sums, no split partials): where tiles of 4 or 3 row blocks x 128 rows give every compute unit work.  Where smaller
// ones would be needed for that (O and down projections of the 8B shape up to 512 rows), the K splits go to
// blocks of their own.
inline bool gemm_whole_k(int M, int N, int K, int epi, bool allow_split) {
  if (M <= 256) return false;
  const GemmPlan p = gemm_plan(N, K, epi == kEpiResidual ? kEpiPartial : epi, allow_split && epi != kEpiSample);
  if (p.kb_per_wave % 4) return false;
  if (epi == kEpiSample) return true;
  const int n_rb = epi == kEpiSwiGLU ? (N >> 4) : (N >> 5), m_tiles = (M + 127) / 128;
  int best = 0, best_cost = 0;
  for (int nb = 4; nb >= 2; --nb) {
    const int blocks = (n_rb + nb - 1) / nb * m_tiles;
    const int cost = (blocks + kComputeUnits - 1) / kComputeUnits * nb;
    if (!best || cost < best_cost) { best = nb; best_cost = cost; }
  }
  return best > 2;
}

struct GemmTile {
  int nb, nw;  // row blocks and waves of a block of gemm_bf16_tile_kernel
};

// The tile of a product of more than 64 rows (K quarters of a multiple of four k blocks).  Figures: the launch by itself, over the weights
// of twelve layers.
//   - Up to 128 rows (one batch tile, HBM bound): 128-row weight tiles where they make 192 blocks or more, 96-row ones where
//     those make a block per compute unit and 128-row ones do not (gate/up at 128 rows 42.9 against 46.0 us, QKV 15.7 against
//     17.9), 64-row ones for the small matrices (O 12.6 against 15.7, down 26.7 against 35.4).
//   - Up to 256 rows: eight waves, so that the weights are read once, by the same rule; matrices with fewer tiles take two
//     batch tiles of four waves (O at 160 / 256 rows 15.0 / 18.2 us, with eight waves 18.5 / 23.8; down 30.0 / 39.2, 39.7 / 49.8).
//   - Beyond: the least time by rounds of blocks.  Four waves have two blocks on a unit, and a last round of one block per
//     unit takes 0.62 of a full one; eight waves have one, and blocks of a last batch tile of up to 128 rows take 0.55 of
//     a full one.  A full round of gate/up takes 58 us with tiles of 3 row blocks x 128 rows, 69 with 4 x 128,
//     57 with 3 x 256 and 63 with 4 x 256 (running sums of the last do not fit the LDS).  At 301 rows this picks 3 x 256 for gate/up (87 us,
//     3 x 128 takes 88, 4 x 128 92, 4 x 256 101), at 512 4 x 128 (112; 114, 120, 123), at 640 4 x 128 (138; 148, 149, 150), at 768
//     3 x 256 (165; 168, 175, 177), at 1024 4 x 256 (193; 207, 214, 231); for down at 256 / 301 / 512 rows 4 x 128 / 4 x 256 / 4 x 256
//     (39 against 50, 48 against 53, 56 against 63).
//   - Sampling beyond 256 rows: 4 x 128 (1 050 us at 700 rows, 4 x 256 1 069: its long epilogue overlaps with the other block).
inline GemmTile gemm_tile(int M, int N, int K, int epi, bool allow_split) {
  const GemmPlan p = gemm_plan(N, K, epi == kEpiResidual ? kEpiPartial : epi, allow_split && epi != kEpiSample);
  const bool whole = gemm_whole_k(M, N, K, epi, allow_split), sums = whole && (p.splits > 1 || epi == kEpiResidual);
  const int n_rb = epi == kEpiSwiGLU ? (N >> 4) : (N >> 5), splits = whole ? 1 : p.splits;
  const auto tiles = [&](int nb) { return (n_rb + nb - 1) / nb * splits; };
  if (M <= 256) {
    const int wide = tiles(4);
    if (wide >= 192) {
      const bool three = epi != kEpiSample && n_rb % 3 == 0 && wide < kComputeUnits && tiles(3) <= kComputeUnits;
      return {three ? 3 : 4, M <= 128 ? 4 : 8};
    }
    return {M > 128 && wide * 2 >= 192 ? 4 : 2, 4};
  }
  if (epi == kEpiSample) return {4, 4};
  const int halves = (M + 127) / 128;
  GemmTile best = {4, 4};
  float best_cost = 0.f;
  for (const GemmTile t : {GemmTile{4, 4}, GemmTile{3, 4}, GemmTile{3, 8}, GemmTile{4, 8}}) {
    if (sums && t.nb == 4 && t.nw == 8) continue;
    float rounds;
    if (t.nw == 4) {
      const int blocks = tiles(t.nb) * halves, left = blocks % (2 * kComputeUnits);
      rounds = (float)(blocks / (2 * kComputeUnits)) + (left == 0 ? 0.f : left <= kComputeUnits ? 0.62f : 1.f);
    } else {
      const int full = tiles(t.nb) * (halves / 2), light = tiles(t.nb) * (halves & 1);
      rounds = full + light <= kComputeUnits ? 1.f : (float)((full + kComputeUnits - 1) / kComputeUnits) + 0.55f * light / kComputeUnits;
    }
    const float cost = rounds * (t.nw == 4 ? (t.nb == 4 ? 69.f : 58.f) : (t.nb == 4 ? 63.f : 57.f));
    if (best_cost == 0.f || cost < best_cost) { best = t; best_cost = cost; }
  }
  return best;
}

}  // namespace rl
