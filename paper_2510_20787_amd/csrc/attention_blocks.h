// Which blocks of 32 keys a wave of the bf16 prefill attention walks.  Plain constexpr C++: the kernel runs it, and a host program
// can walk the same schedule (tests/host_check/attention_blocks_check.cpp).
//
// Block i < n_win holds the keys j_low + 32 * i ..+31, up to the diagonal; block n_win + b the compact slots 32 * b ..+31.  Two
// blocks are a tile, which all waves of the workgroup load together and wait for together: every wave passes the same
// n_tiles() tiles, whatever it sees of them.
//
// What is known of the compact segment (its positions in LDS, the bits below) are the blocks base .. next_base() - 1, 64 of them
// (63 at first where n_win is odd, so that a tile's blocks are known together).  A longer segment is walked group by group.
#pragma once

namespace ltea {

constexpr int BK = 32;   // keys per block

enum : int { kSkip = 0, kPlain = 1, kMasked = 2 };

struct BlockSchedule {
  // of the workgroup
  int window = 0, i_last = 0;        // last query row that exists
  int j_low = 0, n_win = 0;          // j_low may lie before the sequence's start
  int base = 0;                      // first compact block of the group
  int n_blocks = 0;                  // n_win, and the compact blocks up to the last one of the group that some row sees
  // of the wave
  int r0 = 0, r_hi = 0, first_hi = 0;     // first and last row, the last one's first key
  int w_from = 0, w_to = 0, p_from = 0, p_to = 0;   // window blocks that some row sees, and that every row sees whole
  int lim_hi = 0, lim_lo = 0;        // positions that the last and the first row have behind their window
  // Bit b of `ret_any`: some entry of compact block base + b has left the window of the wave's last row; of `ret_all`: every slot
  // of it holds an entry that has left the window of its first row.
  unsigned long long ret_any = 0, ret_all = 0;

  // The workgroup owns the query rows i0 .. i0 + rows - 1 of a sequence of n, the wave the 32 rows from first_row on.
  [[gnu::always_inline]] constexpr BlockSchedule(int i0, int rows, int n, int window_, int first_row)
      : window(window_), r0(first_row), r_hi(first_row + 31) {
    i_last = (i0 + rows < n ? i0 + rows : n) - 1;
    const int j_first = i0 - window + 1 > 0 ? i0 - window + 1 : 0;
    const int j_diag = i0 + ((i_last - i0) & ~(BK - 1));            // the block of the last real query row
    n_win = (j_diag - j_first + BK - 1) / BK + 1;
    j_low = j_diag - BK * (n_win - 1);
    n_blocks = n_win;
    const int first = r0 - window + 1 > 0 ? r0 - window + 1 : 0;
    first_hi = r_hi - window + 1 > 0 ? r_hi - window + 1 : 0;
    w_from = first > j_low ? (first - j_low) / BK : 0;
    w_to = r0 >= n ? 0 : r_hi < j_diag ? (r_hi - j_low) / BK + 1 : n_win;
    p_from = first_hi > j_low ? (first_hi - j_low + BK - 1) / BK : 0;
    p_to = (r0 - j_low) / BK;
    // Rows past the sequence's end see nothing: a wave that counted what they would see took tiles that the other waves do not
    // load and wait for.  (Below every position: the kept entries of a continued prefill have negative ones.)
    lim_hi = r0 < n ? (r_hi < i_last ? r_hi : i_last) - window : -0x7FFFFFFF - 1;
    lim_lo = r0 - window;
  }

  [[gnu::always_inline]] constexpr int n_tiles() const { return (n_blocks + 1) >> 1; }
  [[gnu::always_inline]] constexpr int first_tile() const { return base == 0 ? 0 : (n_win + base) >> 1; }     // of the group
  [[gnu::always_inline]] constexpr int next_base() const { return ((n_win + base + 64) & ~1) - n_win; }

  // What a compact block of which `lowest` and `highest` are the positions (a slot past the last entry: 2^31 - 1) is to the wave
  // and to the workgroup.
  [[gnu::always_inline]] constexpr bool some_row_sees(int lowest) const { return lowest <= lim_hi; }
  [[gnu::always_inline]] constexpr bool every_row_sees(int highest) const { return highest <= lim_lo; }
  [[gnu::always_inline]] constexpr bool workgroup_sees(int lowest) const { return lowest <= i_last - window; }

  // (a compact block has to be of the group)
  [[gnu::always_inline]] constexpr int classify(int i) const {
    if (i < n_win) return i < w_from || i >= w_to ? kSkip : i >= p_from && i < p_to ? kPlain : kMasked;
    if (i >= n_blocks) return kSkip;
    const int b = i - n_win - base;
    if (((ret_any >> b) & 1) == 0) return kSkip;
    return ((ret_all >> b) & 1) != 0 ? kPlain : kMasked;
  }

  // The tile after the last one of those from t on of which the wave sees both blocks; t if it does not see both of t's.
  [[gnu::always_inline]] constexpr int end_of_whole(int t) const {
    const int i = 2 * t;
    if (classify(i) == kSkip) return t;
    int end = w_to;                                  // the first block that the wave does not see
    if (i >= n_win || w_to >= n_win) {
      const int b = i < n_win ? 0 : i - n_win - base;
      const unsigned long long gone = ~(ret_any >> b);
      end = (i < n_win ? n_win : i) + (gone == 0 ? 64 - b : __builtin_ctzll(gone));
      end = end < n_blocks ? end : n_blocks;
    }
    return end >> 1;
  }

  // The first block from i on that needs a mask.
  [[gnu::always_inline]] constexpr int next_masked(int i) const {
    if (i < n_win) return i < p_from || i >= p_to ? i : p_to;      // p_to: the diagonal
    const unsigned long long part = ~(ret_all >> ((i - n_win - base) & 63));
    return part == 0 ? 0x7FFFFFFF : i + __builtin_ctzll(part);
  }
};

}  // namespace ltea
