// How the scoring launches cut a packed batch into workgroups (paper Section 3.1.1): plain host arithmetic, without HIP.
#pragma once
#include <stdint.h>

namespace ltea {

struct ScoreBatch { int32_t n_seqs; int64_t total_tokens; int32_t max_seqlen; int32_t Hkv; };

// Workgroups per head that hold up to `span` consecutive tokens of one sequence: exact for a batch of equal lengths, an upper bound
// otherwise.
inline int64_t score_workgroups(const ScoreBatch& b, int64_t span) {
  return (int64_t)b.n_seqs * b.max_seqlen == b.total_tokens ? (int64_t)b.n_seqs * ((b.max_seqlen + span - 1) / span)
                                                            : b.total_tokens / span + b.n_seqs;
}

// Consecutive tiles per workgroup for a kernel of which `slots` workgroups run at once: the number that makes the launch
// shortest when a workgroup costs its tiles plus about `startup` tiles' worth of start-up and the grid runs in rounds of
// `slots` workgroups.  cost: of the launch, in tiles.
struct GroupPick { int tiles; int64_t cost; };
inline GroupPick pick_group_tiles(const ScoreBatch& b, int tile_tokens, int max_tiles, int startup = 3, int slots = 256) {
  GroupPick best{1, -1};
  for (int g = 1; g <= max_tiles; ++g) {
    const int64_t rounds = (score_workgroups(b, (int64_t)g * tile_tokens) * b.Hkv + slots - 1) / slots;
    const int64_t cost = rounds * (g + startup);
    if (best.cost < 0 || cost < best.cost) best = GroupPick{g, cost};
  }
  return best;
}

// Tiling of the LDS-operand kernel for kernel size ks: waves of 32 tokens per tile, and tiles per workgroup.  single: the form for
// one tile of 128 tokens, whose weights come 64 channels at a time, so that two workgroups and more share a CU; otherwise the
// weights of 128 channels stay in LDS while a group of tiles passes, at k >= 7 with all of a CU's LDS.
//
// k = 1 and 3 have so few weights that the single tiles are never behind (32768 tokens, 32 heads, D = 128: 101 and 118 us against
// 114 and 119).  From k = 5 on long runs of tiles gain from weights that stay (the same tokens, k = 5, 7, 9: 126, 153, 173 us
// against 154, 182, 208) and short sequences from the smaller workgroup: 64 x 100 tokens, 32 heads, D = 128 43, 70, 77 us in
// groups, 38, 45, 52 in single tiles; one sequence of 100 8.8, 10.3, 11.2 and 8.0, 8.9, 9.9.  A round of 512 single tiles took 1.4
// to 1.8 times the unit of pick_group_tiles' cost over these shapes and 64 x 300, 3 x 1000 and 4 x 4096 tokens.
constexpr int kScoreMfmaMaxGroup = 8;
struct ScoreMfmaTiling { int waves, tiles; bool single; };
inline ScoreMfmaTiling score_mfma_tiling(const ScoreBatch& b, int ks) {
  constexpr ScoreMfmaTiling one{4, 1, true};
  if (ks <= 3) return one;
  // a workgroup's start (sequence, weights, first rows) costs about a tile: 4.3 us and 3.7 us per tile of D = 128, k = 5
  const int waves = ks <= 5 ? 4 : 8;
  const GroupPick group = pick_group_tiles(b, 32 * waves, kScoreMfmaMaxGroup, 1, waves == 4 ? 512 : 256);
  const int64_t rounds = (score_workgroups(b, 128) * b.Hkv + 511) / 512;
  return 7 * rounds <= 4 * group.cost ? one : ScoreMfmaTiling{waves, group.tiles, false};
}

}  // namespace ltea
