// The tiling that csrc/score_groups.h picks for batches given on stdin, one "n_seqs total_tokens max_seqlen Hkv kernel" a line:
// prints "waves tiles single" for each.
#include <cstdio>

#include "../../paper_2510_20787_amd/csrc/score_groups.h"

int main() {
  long long total;
  int n_seqs, longest, heads, ks;
  while (std::scanf("%d %lld %d %d %d", &n_seqs, &total, &longest, &heads, &ks) == 5) {
    const ltea::ScoreMfmaTiling t = ltea::score_mfma_tiling(ltea::ScoreBatch{n_seqs, total, longest, heads}, ks);
    std::printf("%d %d %d\n", t.waves, t.tiles, t.single ? 1 : 0);
  }
}
