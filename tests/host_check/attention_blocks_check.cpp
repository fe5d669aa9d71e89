// Walks the block schedule of the bf16 prefill attention (csrc/attention_blocks.h) on the host, the way the kernel's four waves
// do, over random sequences, windows and compact segments in any order.  Checks that all waves pass the same tiles (each one
// waits for the others at every tile), that every (row, key) pair of the set formula is computed exactly once, that a block
// taken without a mask has none to apply, and that a wave without a row computes nothing.  Prints "0 failures" and exits with 0
// if all hold.
#include <cstdio>
#include <cstdint>
#include <algorithm>
#include <random>
#include <vector>

#include "../../paper_2510_20787_amd/csrc/attention_blocks.h"

using namespace ltea;

static long failures = 0, workgroups = 0;
static std::mt19937_64 rng(20787);
static int pick(int lo, int hi) { return lo + (int)(rng() % (uint64_t)(hi - lo + 1)); }

struct Segment {
  std::vector<int> pos;
  int at(int slot) const { return slot < (int)pos.size() ? pos[slot] : 0x7FFFFFFF; }
};

static int highest_or(const Segment& s, int b, bool lowest) {
  int v = s.at(BK * b);
  for (int e = 1; e < BK; ++e) v = lowest ? std::min(v, s.at(BK * b + e)) : std::max(v, s.at(BK * b + e));
  return v;
}

// The wave's bits of the group, and its last block that the workgroup sees.
static void note(BlockSchedule& p, const Segment& s) {
  int seen = 0;
  p.ret_any = p.ret_all = 0;
  for (int b = p.base; b < p.base + 64 && b < p.next_base() && BK * b < (int)s.pos.size(); ++b) {
    const int low = highest_or(s, b, true), high = std::max(0, highest_or(s, b, false));
    if (p.some_row_sees(low)) p.ret_any |= 1ull << (b - p.base);
    if (p.every_row_sees(high)) p.ret_all |= 1ull << (b - p.base);
    if (p.workgroup_sees(low)) seen = b - p.base + 1;
  }
  p.n_blocks = p.n_win + p.base + seen;
}

static void workgroup(int n, int window, int i0, int rows, const Segment& seg, const char* what) {
  ++workgroups;
  long bad = 0;
  int tiles_of[4];
  const int cnt = (int)seg.pos.size();
  for (int wave = 0; wave < 4; ++wave) {
    const int r0 = i0 + (rows == 128 ? 32 * wave : 0);
    BlockSchedule p(i0, rows, n, window, r0);
    // keys of the sequence and slots of the segment that each row has taken
    std::vector<std::vector<int>> key(32, std::vector<int>(n, 0)), slot(32, std::vector<int>(cnt, 0));
    auto visit = [&](int i) {
      const int kind = p.classify(i);
      if (kind == kSkip || r0 >= n) { ++bad; return; }      // a wave without a row has nothing to compute
      for (int r = 0; r < 32; ++r)
        for (int e = 0; e < BK; ++e) {
          const int row = r0 + r;
          if (i < p.n_win) {
            const int j = p.j_low + BK * i + e;
            const bool sees = j >= 0 && j <= row && j > row - window;
            if (row < n && kind == kPlain && !sees) ++bad;
            if (row < n && sees) ++key[r][j];
          } else {
            const int c = BK * (i - p.n_win) + e;
            const bool sees = c < cnt && seg.at(c) <= row - window;
            if (row < n && kind == kPlain && !sees) ++bad;
            if (row < n && sees) ++slot[r][c];
          }
        }
    };
    int settled_at = pick(2, 5), visited = 0, passed = 0;      // blocks by themselves before the reference values are settled
    while (true) {
      note(p, seg);
      const int n_tiles = p.n_tiles();
      if (p.next_base() - p.base > 64 || n_tiles > std::max((p.n_win + p.next_base()) / 2, p.first_tile())) ++bad;
      for (int t = p.first_tile(); t < n_tiles;) {
        const int end = visited >= settled_at ? p.end_of_whole(t) : t;
        if (end > n_tiles) ++bad;
        for (; t < end; ++t, ++passed) {
          const int masked_at = p.next_masked(2 * t);
          for (int i = 2 * t; i < 2 * t + 2; ++i) {
            if (i < masked_at && p.classify(i) != kPlain) ++bad;
            visit(i);
          }
        }
        if (t >= n_tiles) break;
        for (int i = 2 * t; i < 2 * t + 2; ++i)
          if (p.classify(i) != kSkip) { visit(i); ++visited; }
        ++t, ++passed;
      }
      const int next = p.next_base();
      if (BK * next >= cnt) break;
      p.base = next;
    }
    tiles_of[wave] = passed;
    for (int r = 0; r < 32 && r0 + r < n; ++r) {
      for (int j = 0; j < n; ++j) bad += key[r][j] != (j <= r0 + r && j > r0 + r - window);
      for (int c = 0; c < cnt; ++c) bad += slot[r][c] != (seg.pos[c] <= r0 + r - window);
    }
  }
  for (int w = 1; w < 4; ++w) bad += tiles_of[w] != tiles_of[0];
  if (bad) {
    ++failures;
    if (failures <= 10)
      std::printf("FAILED %s: n %d window %d i0 %d rows %d entries %d: tiles %d %d %d %d\n", what, n, window, i0, rows, cnt,
                  tiles_of[0], tiles_of[1], tiles_of[2], tiles_of[3]);
  }
}

// Entries of a sequence of n in some order: 0 ascending, 1 random, 2 descending, 3.. that many interleaved ascending runs.
static Segment segment(int lo, int hi, int m, int order) {
  Segment s;
  std::vector<int> all;
  for (int p = lo; p < hi; ++p) all.push_back(p);
  std::shuffle(all.begin(), all.end(), rng);
  all.resize(std::min<size_t>(all.size(), (size_t)m));
  if (order != 1) std::sort(all.begin(), all.end());
  if (order == 2) std::reverse(all.begin(), all.end());
  if (order >= 3) {
    std::vector<int> runs;
    for (int r = 0; r < order; ++r)
      for (size_t k = r; k < all.size(); k += order) runs.push_back(all[k]);
    all = runs;
  }
  s.pos = all;
  return s;
}

static void all_tiles(int n, int q_begin, int window, const Segment& seg, const char* what) {
  for (int rows : {128, 32})
    for (int i0 = q_begin; i0 < n; i0 += rows) workgroup(n, window, i0, rows, seg, what);
}

int main() {
  // three interleaved runs of the last 96 positions: the blocks at the end of the segment hold only positions that the rows past
  // the sequence's end would see
  all_tiles(277, 0, 96, segment(181, 277, 96, 3), "runs");
  for (int k = 0; k < 3000; ++k) {
    const int n = pick(1, 420), window = pick(1, 200), order = pick(0, 5);
    const int lo = pick(0, 2) == 0 ? std::max(0, n - window - pick(0, 120)) : 0;
    all_tiles(n, 0, window, segment(lo, n, pick(0, 300), order), "prefill");
  }
  // continuations: queries are the last ones, entries of the past have negative positions
  for (int k = 0; k < 1000; ++k) {
    const int window = pick(1, 150), q_begin = window, n = q_begin + pick(1, 200);
    all_tiles(n, q_begin, window, segment(-pick(1, 300), n - window, pick(0, 260), pick(0, 5)), "append");
  }
  // segments of more than 64 blocks
  for (int k = 0; k < 30; ++k) {
    const int n = pick(2100, 4700), window = pick(1, 200);
    const Segment s = segment(0, n, pick(2000, n), pick(0, 5));
    for (int rows : {128, 32})
      for (int m = 0; m < 6; ++m) workgroup(n, window, rows * pick(0, (n - 1) / rows), rows, s, "long");
  }
  std::printf("%ld workgroups, %ld failures\n", workgroups, failures);
  return failures ? 1 : 0;
}
