// Which block of a linear layer a workgroup of a wide pass computes (plain C++: no HIP types).
#pragma once

#include <cstdint>

namespace ssd {

// The blocks that wide_block_kernel is compiled for, feature tiles x row tiles, and what a workgroup is expected to take (us): a step of
// 32 inputs 0.18 and 0.0027 more per tile product (measured at full grids: 4 x 6 tiles 0.20, 8 x 6 0.28 to 0.33, 8 x 8 0.33, 8 x 12 0.42,
// 16 x 12 0.74, 16 x 16 0.85 to 0.95), 1.5 per block, and each k-slice 0.1 and what writing and reading its partial sums costs at 6 TB/s,
// beyond four slices 0.4 more (the residual kernel loads four at a time; with 1 instead, which takes down of 384 rows of the 1B shape from
// eight slices in blocks of 8 x 12 to four in blocks of 8 x 6, rounds of 384 rows take 3 % longer).
// Taken is the cheapest; with one slice and few enough rows that is the smallest block that leaves no workgroup a second one.  Best of a
// sweep, and how much longer a launch with the second best took (2048 inputs, 16384 features): 64 rows 4 x 4, 4 x 6 15 %; 128 rows 4 x 8, 8 x 6
// 18 %; 192 rows 8 x 6, 8 x 8 10 %; 256 rows 8 x 8, 8 x 12 32 %; 384 rows 8 x 12, 16 x 8 6 %; 512 rows 16 x 8, 8 x 8 10 %; 768 rows 16 x 12, 16 x 16
// 4 %; 1020 rows 16 x 16, 16 x 8 23 %.
struct WideBlock { int ft, rt; };
constexpr WideBlock kWideBlocks[] = {{4, 2}, {4, 4}, {4, 6}, {4, 8}, {8, 6}, {8, 8}, {8, 12}, {16, 8}, {16, 12}, {16, 16}, {16, 6}};
constexpr int kNumWideBlocks = sizeof(kWideBlocks) / sizeof(kWideBlocks[0]);   // the last one for the LM head only (288 rows: three groups)
// Gate/up takes all but that one; qkv, o and down no block of 16 x 12 or 16 x 16, which no shape of a fused pass has the features for on
// 256 workgroups (at most 512 tiles of qkv, 128 of o and down in two or more slices).
constexpr int kGateUpBlocks = kNumWideBlocks - 1, kLayerBlocks = 8;

// Rows of partial sums a context has room for, whose wide passes have at most `rows` rows: eight slices of a round's (at most
// `round_rows`), four of a prompt pass's (what eight would write and read again costs more than the larger blocks of a slice save).
constexpr int64_t wide_part_room(int64_t rows, int64_t round_rows, int max_slices) {
  const int64_t round = max_slices * (rows < round_rows ? rows : round_rows), prompt = rows > round_rows ? max_slices / 2 * rows : 0;
  return round > prompt ? round : prompt;
}

struct WideChoice { int block, S; };

// Layers that wide_few_kernel takes instead, over whole sets of 4 feature tiles: row tiles of a group, k-slices and chunks of its ring (0: it
// does not).  Up to 48 rows all of qkv in one turn, and what is short enough of the others.  us that a pass of 8 layers gains (-) or loses
// with it on that layer, blocks alone 268 to 413: width 512 (d_ffn 512, 2048, 8192; 4 to 48 rows) qkv -9 to -16, o -9 to +2, gate/up -12 to +1,
// down -19 to 0; width 1024 (1024, 4096, 8192) qkv -3 to -12, o -9 to 0 up to 32 rows and -1 to +5 beyond, gate/up -9 to +1 at a d_ffn of 1024
// and -2 to +12 above, down -12 to 0 up to 32 rows and -1 to +6 beyond; four layers of width 2048 (2048, 8192) qkv 0 to -8, o -6 to +4, gate/up
// -3 to +6 and +9 to +13, down -6 to +4 and +1 to +3.
constexpr int kFewRows = 48;
enum FewLayer { FEW_QKV, FEW_PART, FEW_GATE_UP };
struct FewChoice { int mtg, S, depth; };
inline FewChoice choose_wide_few(FewLayer layer, int tiles, int k_tiles, int rows, int workgroups, int max_slices, int64_t room) {
  const int row_tiles = (rows + 15) / 16, sets = (tiles + 3) / 4, work = sets * k_tiles;
  if (rows > kFewRows || k_tiles % 16 != 0) return FewChoice{0, 1, 0};
  int S = 1;
  if (layer == FEW_QKV && sets * row_tiles > workgroups) return FewChoice{0, 1, 0};
  if (layer == FEW_GATE_UP && k_tiles > 16 && sets > 64) return FewChoice{0, 1, 0};
  if (layer == FEW_PART) {
    if (work > (rows <= 32 ? 4096 : 2048)) return FewChoice{0, 1, 0};
    for (S = max_slices; S > 1; S /= 2)                       // as many slices as leave every workgroup one pair
      if (sets * S <= workgroups && (int64_t)S * rows <= room && k_tiles % (16 * S) == 0) break;
  }
  // qkv: a row tile per workgroup, so that more of them share the weights
  const int mtg = layer == FEW_QKV || (layer == FEW_PART && row_tiles == 1) ? 1 : row_tiles <= 2 ? 2 : 3;
  return FewChoice{mtg, S, k_tiles / (4 * S) % 8 == 0 ? 8 : 4};   // (a wavefront's quarter of a slice is whole turns of the ring)
}

// tiles: 16-feature tiles of the layer; k_tiles: of its reduction dimension; blocks: how many of the list it may take; room: rows of
// partial sums there is memory for (0: no k-slices); out_width: features of such a row.
inline WideChoice choose_wide_block(int tiles, int k_tiles, int rows, int workgroups, int blocks, int max_slices, int64_t room, int out_width) {
  const int per_xcd = workgroups / 8, row_tiles = (rows + 15) / 16;
  WideChoice best{0, 1};
  float best_us = 0.0f;
  for (int S = 1; S <= (room > 0 ? max_slices : 1); S *= 2) {
    if (k_tiles % (2 * S) != 0 || (S > 1 && (int64_t)S * rows > room)) break;   // whole pairs of steps per slice
    for (int i = 0; i < blocks; ++i) {
      const int area = kWideBlocks[i].ft * kWideBlocks[i].rt, ys = 8 / S;       // dies that share a slice
      const int sets = (tiles + kWideBlocks[i].ft - 1) / kWideBlocks[i].ft, groups = (row_tiles + kWideBlocks[i].rt - 1) / kWideBlocks[i].rt;
      const int turns = ((sets + ys - 1) / ys * groups + per_xcd - 1) / per_xcd;
      float us = (float)turns * ((float)(k_tiles / S) * (0.18f + 0.0027f * (float)area) + 1.5f);
      if (room > 0) us += (float)S * (0.1f + (float)rows * (float)out_width * 8.0f / 6e6f) + (S > 4 ? 0.4f : 0.0f);
      if ((S == 1 && i == 0) || us < best_us) {
        best_us = us;
        best = WideChoice{i, S};
      }
    }
  }
  return best;
}

}  // namespace ssd
