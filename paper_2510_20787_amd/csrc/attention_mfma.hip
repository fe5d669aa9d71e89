// Prefill attention over window + retained set (paper Section 3.1.3) on bf16 MFMA for gfx950.
//
// Flash-attention-style tiling, two stages per query tile as in the paper's description: stage 1 walks blocks of 32 keys
// of the original K/V inside the tile's window range, stage 2 walks blocks of 32 slots of the compact retained segment with a
// per-row mask "position <= i - window" (so entries still inside a query's window are never counted twice).  Two blocks
// make a tile, which is what is loaded at once.
//
// Work split: one workgroup = 128 consecutive queries of one (sequence, query head), 4 waves each owning a block
// of 32 queries; or, for grouped-query shapes, the same 32 queries of four query heads that share a KV head, one
// head per wave.  MFMA shapes (v_mfma_f32_32x32x16_bf16, wave64):
//   S^T[key, query] = K[key, :] . Q[query, :]   A = K tile rows from LDS, B = Q fragment held in registers
//   O^T[d, query]  += V^T[d, key] . P^T[key, query]   A = V^T fragments from LDS, B = P^T straight from S^T's
//                                                     accumulator registers (no shuffle, no LDS round trip)
// In the 32x32 accumulator layout a lane owns one query column, so the softmax statistics are per-lane scalars
// (the two lanes sharing a query keep separate partial sums and meet once, in the epilogue).  The contraction index of
// the second product is the key index; the rows of the K tile are fed to the first MFMA in a permuted
// order so that each lane's eight P values per MFMA are eight consecutive keys.  V stays row-major in LDS
// and its A operand (eight consecutive keys of one column per lane) comes out of the transposing LDS load
// ds_read_b64_tr_b16, two per MFMA; the tile's 64-byte chunks are XOR-swizzled so that those loads spread over the
// 64 banks without padding.
// K and V tiles are double-buffered in LDS and come there straight from global memory, one barrier per tile (three
// workgroups share a CU at D = 64, two at D = 128).  There is no running maximum: a row's exponentials are taken
// relative to the maximum of the first two blocks in which it sees a key (the result does not depend on that reference
// value as long as the exponentials stay in range; a workgroup whose row sums leave the range repeats its tiles with
// the exact running maximum in every block), which keeps the row-maximum reduction and the accumulator rescale off the
// common path.
//
// A workgroup's blocks are its window's, aligned to its query rows, then those of the compact segment that some row of it
// sees; a wave leaves out the ones that none of its rows sees.  Aligned to the rows, a window of a multiple of 32 costs its
// blocks plus one, two of them masked; tiles of 64 keys on a fixed grid cost up to three blocks more, and blocks of the
// segment that lie in the future of all rows (half of them on average) were loaded and waited for.  Window blocks go in
// ascending order: neighbouring workgroups, which start one after the other, then meet in the L2 (from the diagonal down
// 4.0 GB instead of 1.4 came from beyond it for 32768 tokens x 32 heads of D = 128).
//
// What bounds it: at D = 128 the clock that power leaves (1.80 GHz of 2.4, as for a bare loop of matrix instructions on normally
// distributed operands, which reaches 1.84 PFLOP/s there and 2.45 on zeros) and a matrix pipe that is busy in 58 % of those
// clocks; at D = 64 the issue of a wave's instructions (a matrix instruction holds it for 16 clocks of its 32, an exponential
// for 8, others for 4) and the start of a workgroup (7000 to 8000 of 44000 to 51000 clocks: sequence, count, positions, first
// tile).  Kernel time, tiles on the fixed grid and this form in turn on one box:
// 32768 tokens x 32 heads of D = 128 1435 -> 1298 us; 4 x 4096 tokens, 32 query heads on 8 of D = 64 166 -> 151 us, 16 heads
// of D = 64 67.9 -> 63.3 us; 777 tokens, 32 on 8 heads 16.0 -> 13.5 us.  Windows of up to 64 keys on one head per workgroup lose:
// a wave's few blocks then run by themselves, the operands of the second waiting for the first (4 x 4096 tokens, 16 heads, 64
// kept: D = 64, window 16 36.7 -> 38.7 us, window 64 37.0 -> 38.3; D = 128, window 48 67.0 -> 68.5, window 16 67.7 -> 63.9).
// Neither one block for the reference values (38.7 -> 38.8 us at window 16) nor an even number of window blocks (38.2 there, but
// 151 -> 152 us for the 4 x 4096 tokens above and 13.6 -> 14.9 for the 777) changes that.
// Tried and not kept: the products of one block beside the scores of the next across tiles (same speed, and every first and
// last block of a wave runs by itself); 64 queries per wave at D = 64 (half the operand reads, but 47 registers spilled: 192 us
// against 162); blocks that run by themselves with all their operands requested ahead (windows of up to 128 keys 1 to 2 %
// slower).
#include <type_traits>

#include "attention_blocks.h"
#include "ltea_common.h"
#include "ltea_kernels.h"
#include "mfma_tiles.h"
#include "score_dma.h"

namespace ltea {
namespace {

constexpr int BN = 64;   // keys per tile: two blocks
constexpr int kThreads = 256;
constexpr int kPosLds = 64 * BK;   // positions of the compact segment kept in LDS (longer segments: group by group)
constexpr float kBig = 1.8446744e19f;  // 2^64: a row sum above this (or not a number) sends the workgroup through its tiles again

template <int D> struct Geo {
  static constexpr int BM = 128;                // query rows per workgroup
  static constexpr int PPR = D / 8;             // 16-byte pieces per row
  static constexpr int RPI = 64 / PPR;          // rows per wave load instruction
  static constexpr int IPB = BK / RPI / 4;      // load instructions per wave and block of keys (or values)
  static constexpr int OS = D + 8;              // epilogue staging row stride (elements)
  static constexpr int kTile = BN * D;          // elements of one tile, rows unpadded; K tile then V tile per buffer
  static constexpr int kBuf = 2 * kTile;
  static constexpr int kLds = 4 * kTile > BM * OS ? 4 * kTile : BM * OS;
};

// Which 16-byte piece of its row a K tile row keeps at slot p (p ^ term): the row reads of 16 consecutive lanes (16 rows at
// one piece) then cover all 64 banks.
template <int D> __device__ __forceinline__ int piece_swizzle(int row) { return D == 64 ? ((row >> 1) & 7) : (row & 15); }

// HW = query heads per workgroup.  1: the four waves take four consecutive blocks of 32 query positions of one head.
// 4 (grouped-query shapes with a multiple of four query heads per KV head): the four waves take the SAME 32
// positions of four query heads that share the KV head.  The K/V tiles are shared either way, but with HW = 4 every wave
// sees the same window, so a block is plain, masked or out of reach for all four at once (with HW = 1 the waves' windows
// are shifted by 32 positions each, the workgroup's key range is 96 positions longer, and waves wait for each other at
// the tile barrier).
template <int D, int HW>
__global__ void __launch_bounds__(kThreads, D == 64 ? 3 : 2)
attention_mfma_kernel(const bf16_t* __restrict__ q, int64_t q_st, int64_t q_sh, const bf16_t* __restrict__ k,
                      const bf16_t* __restrict__ v, int64_t kv_st, int64_t kv_sh, const int32_t* __restrict__ cu,
                      int n_seqs, int tiles_upper, int n_work, int Hq, int Hkv, int window, int budget,
                      float scale_log2e, const bf16_t* __restrict__ k_ret, const bf16_t* __restrict__ v_ret,
                      const int32_t* __restrict__ ret_pos, const int32_t* __restrict__ ret_count,
                      bf16_t* __restrict__ out, const int32_t* __restrict__ kv_start,
                      const int32_t* __restrict__ kv_len, float* __restrict__ lse, int64_t lse_stride) {
  using G = Geo<D>;
  constexpr int BM = G::BM, kTile = G::kTile, kBuf = G::kBuf;
  constexpr int BMQ = BM / HW;     // query positions per workgroup (BM = rows of all its waves)
  static_assert(HW == 1 || HW == 4, "one head, or one head per wave");
  __shared__ __align__(1024) bf16_t lds[G::kLds];
  __shared__ __align__(256) int pos_lds[kPosLds];
  __shared__ int redo_flag;

  // ---- which (query head, sequence, query tile) is this workgroup? ------------------------------------
  // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of work items so
  // that neighbouring query tiles of one head (which share most of their keys) meet in the same L2.  When the heads
  // divide evenly over the XCDs, an XCD takes whole heads and walks them tile by tile, heads fastest, long tiles first:
  // the first tiles of every sequence, whose window is still filling, come last and fill the gaps when the grid drains.
  const int per_xcd = (n_work + 7) / 8;
  const int work = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (work >= n_work) return;
  int unit, flat_tile;                      // unit = query head (HW = 1) or group of HW query heads
  const int units = Hq / HW;
  const bool whole_heads = units % 8 == 0;
  if (whole_heads) {
    const int hpx = units / 8, in_xcd = blockIdx.x / 8;      // per_xcd == hpx * tiles_upper
    unit = (blockIdx.x % 8) * hpx + in_xcd % hpx;
    flat_tile = in_xcd / hpx;
  } else {
    unit = work / tiles_upper;
    flat_tile = work - unit * tiles_upper;
  }
  // cu packs the query / output rows.  Normally it packs the keys as well; with kv_start / kv_len given, the keys
  // of sequence s are rows kv_start[s] .. kv_start[s] + kv_len[s] - 1 of k / v and the queries are the last
  // cu[s+1] - cu[s] positions of that key sequence (continuation of a prefill).
  int tile, s, n, lo_q;
  if (whole_heads && kv_start == nullptr) {
    if (!locate_tile_late_first(cu, n_seqs, BMQ, (window + BMQ - 1) / BMQ, flat_tile, s, tile, lo_q, n)) return;
  } else {
    if (!locate_tile(cu, n_seqs, BMQ, flat_tile, s, tile, lo_q, n)) return;
  }
  int64_t lo = lo_q;
  int q_begin = 0;
  if (kv_start != nullptr) {
    const int nq = n;
    lo = kv_start[s];
    n = kv_len[s];
    q_begin = n - nq;
  }
  const int h = (unit * HW) / (Hq / Hkv);
  const int64_t head = (int64_t)s * Hkv + h;
  const int i0 = q_begin + tile * BMQ;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ql = lane & 31, hb = lane >> 5;
  const int hq = HW == 1 ? unit : unit * HW + wv;                 // this wave's query head
  const int r0 = i0 + (HW == 1 ? 32 * wv : 0);               // first query row of this wave
  BlockSchedule plan(i0, BMQ, n, window, r0);
  const int i_last = plan.i_last, j_low = plan.j_low, n_win = plan.n_win, first_hi = plan.first_hi;

  // ---- per-thread load addressing: buffer loads with 32-bit byte offsets; rows outside the sequence (or past ret_count in
  // the compact segment) are out of the descriptor's range and read as zeros ------------------------------------------
  const uint32_t row_bytes = (uint32_t)kv_st * 2u;
  const uint32_t win_bytes = (uint32_t)(n - 1) * row_bytes + (uint32_t)(D * 2);
  const u32x4 rs_k = make_raw_rsrc(k + lo * kv_st + (int64_t)h * kv_sh, win_bytes);
  const u32x4 rs_v = make_raw_rsrc(v + lo * kv_st + (int64_t)h * kv_sh, win_bytes);
  u32x4 rs_kr, rs_vr;          // set once the count has arrived
  int cnt = 0;
  const int32_t* const head_pos = ret_pos + head * budget;

  // ---- global -> LDS: a wave instruction fills RPI rows (1 KB) of one tile; instruction wv + 4*i.  The tiles are swizzled
  // by which piece a lane fetches: K for the row reads, V (its 64-byte chunks) for the transposing reads.  The swizzle terms
  // of a lane's rows do not depend on i.
  const int ld_row = G::RPI * wv + lane / G::PPR, ld_slot = lane % G::PPR;       // + 4 * RPI * i
  const uint32_t ld_k = (uint32_t)(ld_slot ^ piece_swizzle<D>(ld_row)) * 16u;
  const uint32_t ld_v = (uint32_t)((((ld_slot >> 2) ^ chunk_swizzle<D>(ld_row)) << 2) | (ld_slot & 3)) * 16u;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  auto load_rows = [&](u32x4 rk, u32x4 rv, uint32_t dst, uint32_t off, uint32_t step, const int from, const int to) __attribute__((always_inline)) {
#pragma unroll
    for (int x = from; x < to; ++x) {
      dma16(rk, dst + (uint32_t)(x * 4096), off + (uint32_t)x * step + ld_k);
      dma16(rv, dst + (uint32_t)(kTile * 2 + x * 4096), off + (uint32_t)x * step + ld_v);
    }
  };
  auto load_tile = [&](int t) __attribute__((always_inline)) {
    const uint32_t dst = lds_base + (uint32_t)((t & 1) * kBuf * 2 + wv * 1024);
    const uint32_t win_off = (uint32_t)(j_low + BN * t + ld_row) * row_bytes, ret_off = (uint32_t)(BN * t - BK * n_win + ld_row) * (uint32_t)(D * 2);
    const uint32_t win_step = (uint32_t)(4 * G::RPI) * row_bytes, ret_step = (uint32_t)(4 * G::RPI) * (uint32_t)(D * 2);
    if (2 * t + 1 < n_win) load_rows(rs_k, rs_v, dst, win_off, win_step, 0, 2 * G::IPB);
    else {
      if (2 * t < n_win) load_rows(rs_k, rs_v, dst, win_off, win_step, 0, G::IPB);
      else load_rows(rs_kr, rs_vr, dst, ret_off, ret_step, 0, G::IPB);
      load_rows(rs_kr, rs_vr, dst, ret_off, ret_step, G::IPB, 2 * G::IPB);
    }
  };

  // ---- Q fragments (B operand of S^T): lane holds Q[row][16*ks + 8*hb .. +7] for its row ------------
  bf16x8 qreg[D / 16];
  const int qi = r0 + ql;
  const int qc = qi < n ? qi : n - 1;
  const bf16_t* qrow = q + (int64_t)(lo_q + qc - q_begin) * q_st + (int64_t)hq * q_sh;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8*>(qrow + 16 * ks + 8 * hb);

  // operand load offsets inside a tile buffer (elements).  K: MFMA row ql carries block row kr; its pieces 2*ks + hb.
  const int k_row = tile_row_of_mfma_row(ql);
  const int k_off0 = k_row * D + ((piece_swizzle<D>(k_row) ^ hb) << 3);         // ^ (16 * ks)
  // V operand through the transposing LDS load: in each group of 16 lanes, lane j points at the four columns
  // d0 + 4*(j%4).. of key row kbase + j/4, and receives column d0 + j of the four keys kbase..kbase+3.
  const int tr_key = 8 * hb + ((lane & 15) >> 2);           // + 16*kk (+ 4 for the upper half)
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);  // + 32*db, inside one 64-byte chunk
  const int tr_swz = chunk_swizzle<D>(tr_key);                  // unchanged by adding multiples of 4 to the key
  const int a_v_off = kTile + tr_key * D + tr_col;
  constexpr int NK = D / 16, ND = D / 32;
  // operands of block kb of the tile in buffer `par`: K by contraction step, V in the order (kk, db)
  auto k_op = [&](int par, int kb, int ks) __attribute__((always_inline)) {
    return *reinterpret_cast<const bf16x8*>(lds + par * kBuf + (k_off0 ^ (16 * ks)) + BK * D * kb);
  };
  auto v_op = [&](int par, int kb, int i) __attribute__((always_inline)) {
    return load_transposed(lds + par * kBuf + a_v_off + BK * D * kb + (((i % ND) ^ tr_swz) << 5) + 16 * (i / ND) * D, D);
  };

  // ---- which blocks of the compact segment does this wave see? --------------------------------------------------
  // The group's positions are in LDS (slots past the last entry as 2^31 - 1): 64 blocks.  A longer segment is walked in groups
  // of them: its positions arrive with the group's first tile, and a group that nobody sees costs that one wait.  (Positions
  // read where they were needed, a block at a time, were slower than a load of them with every tile: 2 x 8192 tokens, 16 heads
  // of D = 64 on 4000 entries 228 us with every tile, 292 block by block, 196 in groups; 32768 tokens, 8 heads on 31000 entries
  // 1398, 2079 and 1194 us.)
  auto load_positions = [&]() __attribute__((always_inline)) {
    const int from = BK * plan.base, left = cnt - from, n_lds = left < kPosLds ? (left + BK - 1) & ~(BK - 1) : kPosLds;
#pragma unroll 2
    for (int i = tid; i < n_lds; i += kThreads) pos_lds[i] = i < left ? head_pos[from + i] : 0x7FFFFFFF;
  };
  auto note_blocks = [&]() __attribute__((always_inline)) {
    // lane b looks at block base + b: 16-byte pieces in an order that spreads 16 lanes over all banks
    int lowest = 0x7FFFFFFF, highest = 0;
#pragma unroll 2
    for (int c = 0; c < 8; ++c) {
      const int4 x = *reinterpret_cast<const int4*>(&pos_lds[BK * lane + 4 * ((c + (lane >> 1)) & 7)]);
      lowest = min(min(lowest, x.x), min(min(x.y, x.z), x.w));
      highest = max(max(highest, x.x), max(max(x.y, x.z), x.w));
    }
    const int b = plan.base + lane;
    const bool there = BK * b < cnt && b < plan.next_base();
    plan.ret_any = __builtin_amdgcn_ballot_w64(there && plan.some_row_sees(lowest));
    plan.ret_all = __builtin_amdgcn_ballot_w64(there && plan.every_row_sees(highest));
    const unsigned long long wg = __builtin_amdgcn_ballot_w64(there && plan.workgroup_sees(lowest));
    plan.n_blocks = n_win + plan.base + (wg == 0 ? 0 : 64 - __builtin_clzll(wg));
  };

  // ---- softmax state (per lane = per query; the two lane halves keep separate partial sums) ------
  float m_run, l_part;
  // Row sums of the tiles that are interleaved, on the matrix pipe: v_mfma_f32_16x16x32_bf16 reads a P operand of the value product
  // as 16 columns of which lane groups 0, 2 hold queries 0..15 and groups 1, 3 queries 16..31.  With ones in the rows whose
  // lowest bit is the group's, register 0 of every lane is the sum of query lane%16 and register 1 that of query
  // 16 + lane%16.  (A v_dot2c_f32_bf16 waits for the matrix instruction in flight and holds back the next one.)  A sum that
  // is not finite reaches its neighbour's through 0 * inf, so the repeated pass does not use it.
  f32x4 l_mat;
  bf16x8 sum_rows;
  {
    const bf16_t one = static_cast<bf16_t>(((lane ^ (lane >> 4)) & 1) == 0 ? 1.0f : 0.0f);
#pragma unroll
    for (int e = 0; e < 8; ++e) sum_rows[e] = one;
  }
  int raised = 0;              // blocks whose maximum went into the reference values
  bool all_have_m = false;     // wave-uniform: every row of the wave has a reference value (m_run finite) from two blocks
  bool exact_pass = false;     // workgroup-uniform: second run over the tiles, with the running maximum in every block
  f32x16 o[ND];
  auto reset_rows = [&]() __attribute__((always_inline)) {
    all_have_m = false;
    raised = 0;
    m_run = -INFINITY;
    l_part = 0.f;
    l_mat = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int db = 0; db < ND; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  };
  auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
  auto pin = [](bf16x8& x) {
    u32x4 w = __builtin_bit_cast(u32x4, x);
    asm volatile("" : "+v"(w));
    x = __builtin_bit_cast(bf16x8, w);
  };

  // Scores of block i to -inf where the query does not see the key; register r is block key 16*(r/8) + 8*hb + r%8.
  // (The wait is for the matrix instructions before: the branches below must not come between them and the reads.)
  auto apply_mask = [&](int i, f32x16& x) __attribute__((always_inline)) {
    asm volatile("s_nop 15\n\ts_nop 7" : "+v"(x));
    if (i < n_win) {
      const int j0 = j_low + BK * i;
      if (j0 + BK - 1 > r0) {                                       // causal: j <= query (rows past n see zeros)
        const int c_hi = r0 + ql - j0 - 8 * hb;
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = (16 * (r / 8) + r % 8 <= c_hi) ? x[r] : -INFINITY;
      }
      if (j0 < first_hi) {                                          // window and sequence start: j >= max(query - window + 1, 0)
        const int qi = r0 + ql;
        const int c_lo = (qi - window + 1 > 0 ? qi - window + 1 : 0) - j0 - 8 * hb;
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = (16 * (r / 8) + r % 8 >= c_lo) ? x[r] : -INFINITY;
      }
    } else if (((plan.ret_all >> (i - n_win - plan.base)) & 1) == 0) {
      const int* pos = pos_lds + BK * (i - n_win - plan.base) + 8 * hb;
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = pos[16 * (r / 8) + r % 8] <= r0 + ql - window ? x[r] : -INFINITY;
    }
  };
  // The reference value m of a row (probabilities are exp2(score - m)) only has to keep the exponentials in range,
  // so it is not the running maximum: a row takes the maximum of the first two blocks and keeps it (l is then at least the 1
  // of those, and the softmax is the same function of the scores for any m).  Scores that later exceed m by more than the
  // exponent range allows show up as a huge or non-finite row sum when the tiles are done; the workgroup then runs its
  // tiles a second time with the exact running maximum in every block.
  auto raise_reference = [&](const f32x16& x) __attribute__((always_inline)) {
    float mx = fmaxf(x[0], x[1]);
#pragma unroll
    for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, x[r]), x[r + 1]);
    mx = pair_max(mx);
    const float m_new = fmaxf(m_run, mx * scale_log2e);
    // nothing visible so far and nothing now: m stays -inf, and the factor must not become exp2(nan)
    const float a = (m_new == m_run) ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
    const bool none = m_run == -INFINITY;
    m_run = m_new;
    l_part *= a;
    // A row that has seen nothing has nothing to scale: the first block waits for no accumulator.  (Short windows feel it: 4 x 4096
    // tokens, 16 heads of D = 128, window 16 55.6 -> 54.4 us.)
    if (__builtin_amdgcn_ballot_w64(a != 1.0f && !none) != 0ull) {
#pragma unroll
      for (int db = 0; db < ND; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= a;
    }
    ++raised;
    all_have_m = raised >= 2 && __builtin_amdgcn_ballot_w64(m_new == -INFINITY) == 0ull;
  };

  // A tile of which the wave sees both blocks, once the reference values are settled.  A wave issues in order and a matrix
  // instruction holds the issue for 16 clocks and the matrix pipe for 32: vector instructions placed behind it run in the
  // time that is left, those behind the last one of a row of matrix instructions do not.  So each instruction of block 1's
  // scores and of block 0's value product is followed by its share of the other block's exponentials.
  auto tile_interleaved = [&](auto par, auto MASKED, int t) __attribute__((always_inline)) {
    constexpr int EPM = 16 / NK, HALF = NK / 2;     // operands are read HALF instructions ahead: further ahead spills
    float e[16];
    auto exp_part = [&](int i, const f32x16& x) __attribute__((always_inline)) {
#pragma unroll
      for (int r = EPM * i; r < EPM * (i + 1); ++r) {
        e[r] = __builtin_amdgcn_exp2f(fmaf(x[r], scale_log2e, -m_run));
        asm volatile("" : "+v"(e[r]));      // here, not next to its first use
      }
    };
    auto pack_part = [&](int i, bf16x8 (&p)[2]) __attribute__((always_inline)) {      // of the step before
#pragma unroll
      for (int r = EPM * i; r < EPM * (i + 1); ++r) p[r / 8][r % 8] = static_cast<bf16_t>(e[r]);
    };
    auto product = [&](int i, const bf16x8& a, const bf16x8 (&p)[2]) __attribute__((always_inline)) {
      o[i % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p[i / ND], o[i % ND], 0, 0, 0);
      if (i % ND == ND - 1) l_mat = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sum_rows, p[i / ND], l_mat, 0, 0, 0);
    };
    f32x16 s0, s1;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s0[r] = 0.f; s1[r] = 0.f; }
    bf16x8 p0[2], p1[2], ka[NK], kb[NK], va[NK], vb[NK];
#pragma unroll
    for (int i = 0; i < NK; ++i) ka[i] = k_op(par, 0, i);
    fence();
#pragma unroll
    for (int i = 0; i < NK; ++i) {                       // scores of block 0
      pin(ka[i]);
      s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i], qreg[i], s0, 0, 0, 0);
      if (i >= HALF) kb[i - HALF] = k_op(par, 1, i - HALF);
      fence();
    }
    if constexpr (decltype(MASKED)::value) apply_mask(2 * t, s0);
#pragma unroll
    for (int i = 0; i < NK; ++i) {                       // scores of block 1 / softmax of block 0
      pin(kb[i]);
      s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[i], qreg[i], s1, 0, 0, 0);
      if (i < HALF) kb[i + HALF] = k_op(par, 1, i + HALF);
      else va[i - HALF] = v_op(par, 0, i - HALF);
      exp_part(i, s0);
      if (i > 0) pack_part(i - 1, p0);
      fence();
    }
    pack_part(NK - 1, p0);
    fence();
    if constexpr (decltype(MASKED)::value) apply_mask(2 * t + 1, s1);
#pragma unroll
    for (int i = 0; i < NK; ++i) {                       // value products of block 0 / softmax of block 1
      pin(va[i]);
      product(i, va[i], p0);
      if (i < HALF) va[i + HALF] = v_op(par, 0, i + HALF);
      else vb[i - HALF] = v_op(par, 1, i - HALF);
      exp_part(i, s1);
      if (i > 0) pack_part(i - 1, p1);
      fence();
    }
    pack_part(NK - 1, p1);
    fence();
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      if (i < HALF) vb[i + HALF] = v_op(par, 1, i + HALF);
      pin(vb[i]);
      product(i, vb[i], p1);
      fence();
    }
    fence();
  };
  // One block by itself: the first ones (reference values), tiles of which the wave sees one block, the repeated pass.
  auto block_general = [&](int i) __attribute__((always_inline)) {
    const int par = (i >> 1) & 1, kb = i & 1;
    f32x16 x;
    bf16x8 p[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
      const bf16x8 a = k_op(par, kb, ks);
      x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], x, 0, 0, 0);
    }
    apply_mask(i, x);
    if (!all_have_m || exact_pass) raise_reference(x);
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r / 8][r % 8] = static_cast<bf16_t>(__builtin_amdgcn_exp2f(fmaf(x[r], scale_log2e, -m_use)));
    pin(p[0]);
    pin(p[1]);
    // row sum from the rounded probabilities: the denominator then matches the P that the product consumes
    float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      sum0 += static_cast<float>(p[r / 8][r % 8]);
      sum1 += static_cast<float>(p[r / 8][r % 8 + 1]);
    }
    l_part += sum0 + sum1;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
      const bf16x8 a = v_op(par, kb, j);
      o[j % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p[j / ND], o[j % ND], 0, 0, 0);
    }
  };

  if (tid == 0) redo_flag = 0;
  if (n_win >= 2) load_tile(0);      // of the window only: does not wait for the count of the compact segment's entries
  cnt = __builtin_amdgcn_readfirstlane(budget > 0 && i_last - window >= 0 ? ret_count[head] : 0);
  rs_kr = make_raw_rsrc(k_ret + head * budget * D, (uint32_t)cnt * (uint32_t)(D * 2));
  rs_vr = make_raw_rsrc(v_ret + head * budget * D, (uint32_t)cnt * (uint32_t)(D * 2));
  load_positions();
  if (n_win < 2) load_tile(0);
  reset_rows();
  auto tile_done = [&]() __attribute__((always_inline)) {
    wait_loads();
    __syncthreads();   // tile t + 1 is in LDS; everyone is done with tile t
  };
  // One loop over the groups and the repeated pass, with one place that starts a group: what the prologue needs (counts, base
  // addresses) then does not live through the tiles.  No vector register and at most two scalar ones (at D = 128) are spilled; with
  // the prologue inside a loop over the passes 15 to 25 were, and a workgroup waited for one argument more (4 x 4096 tokens, 16
  // heads of D = 64, window 96, nothing kept: 37.8 -> 35.2 us).
#pragma unroll 1
  while (true) {       // window and first group of the compact segment, further groups of it; perhaps all of it once more
    tile_done();       // the group's first tile and its positions
    plan.n_blocks = n_win;
    if (cnt > 0) note_blocks();
    const int n_tiles = plan.n_tiles();
#pragma unroll 1
    for (int t = plan.first_tile(); t < n_tiles;) {
      // tiles from t on of which the wave sees both blocks
      const int t_end = __builtin_amdgcn_readfirstlane(all_have_m && !exact_pass ? plan.end_of_whole(t) : t);
      int masked_at = __builtin_amdgcn_readfirstlane(plan.next_masked(2 * t));
      if (t < t_end) {
#pragma unroll 1
        do {
          // up to the next one with a mask
          int t_plain = masked_at >> 1;
          t_plain = t_plain < t_end ? t_plain : t_end;
          if (t < t_plain) {
#pragma unroll 1
            while (true) {
              if ((t & 1) == 0) {
                if (t + 1 < n_tiles) load_tile(t + 1);      // everyone is done with tile t - 1, whose buffer this is
                tile_interleaved(std::integral_constant<int, 0>{}, std::false_type{}, t);
                tile_done();
                if (++t == t_plain) break;
              }
              if (t + 1 < n_tiles) load_tile(t + 1);
              tile_interleaved(std::integral_constant<int, 1>{}, std::false_type{}, t);
              tile_done();
              if (++t == t_plain) break;
            }
          }
          t = __builtin_amdgcn_readfirstlane(t);
          if (t < t_end) {
            if (t + 1 < n_tiles) load_tile(t + 1);
            tile_interleaved(t & 1, std::true_type{}, t);
            tile_done();
            ++t;
            masked_at = __builtin_amdgcn_readfirstlane(plan.next_masked(2 * t));
          }
        } while (t < t_end);
      }
      t = __builtin_amdgcn_readfirstlane(t);
      if (t < n_tiles && (t_end <= t)) {
        if (t + 1 < n_tiles) load_tile(t + 1);
#pragma unroll 1
        for (int i = 2 * t; i < 2 * t + 2; ++i)
          if (__builtin_amdgcn_readfirstlane(plan.classify(i)) != kSkip) block_general(i);
        tile_done();
        ++t;
      }
    }
    plan.base = plan.next_base();
    if (BK * plan.base >= cnt) {
      if (exact_pass) break;
      // did a row's reference value fall so far below its scores that its sums left the range?
      const bool bad = !(l_part <= kBig) || !(l_mat[0] <= kBig) || !(l_mat[1] <= kBig);
      if (__builtin_amdgcn_ballot_w64(bad) != 0ull && lane == 0) redo_flag = 1;
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(redo_flag) == 0) break;
      exact_pass = true;
      plan.base = 0;
      reset_rows();
    }
    __syncthreads();   // everyone is done with the tile buffers and has looked at the positions
    load_tile(plan.first_tile());
    load_positions();
  }

  // ---- epilogue: normalise, stage through LDS, store rows coalesced -------------------------------------------
  __syncthreads();  // tile buffers are free
  const float l_row = pair_sum(l_part) + ((lane & 16) != 0 ? l_mat[1] : l_mat[0]);
  const float inv = 1.0f / l_row;
  if (lse != nullptr && hb == 0) {
    // natural-log normaliser of the scaled scores (m_run is kept in the base-2 domain); wanted by a backward pass
    const int row = (HW == 1 ? 32 * wv : 0) + ql;
    if (i0 + row < n) lse[(int64_t)hq * lse_stride + lo_q + i0 + row - q_begin] = (m_run + __log2f(l_row)) * 0.6931471805599453f;
  }
  bf16_t* orow = lds + (32 * wv + ql) * G::OS + 4 * hb;
#pragma unroll
  for (int db = 0; db < ND; ++db)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      bf16x4 w4;
#pragma unroll
      for (int e = 0; e < 4; ++e) w4[e] = static_cast<bf16_t>(o[db][4 * g4 + e] * inv);
      *reinterpret_cast<bf16x4*>(orow + 32 * db + 8 * g4) = w4;
    }
  __syncthreads();
  {
    // staging row = 32*wave + position block: with HW = 1 all rows are positions of one head, with HW = 4 the
    // wave index is the head inside the group
    bf16_t* obase = out + ((int64_t)(lo_q + i0 - q_begin) * Hq + unit * HW) * D;
    const int64_t orow_stride = (int64_t)Hq * D;
    constexpr int kRowsPerPass = kThreads / G::PPR;
#pragma unroll
    for (int p = 0; p < BM / kRowsPerPass; ++p) {
      const int row = p * kRowsPerPass + tid / G::PPR;
      const int prow = HW == 1 ? row : row % (32), hd = HW == 1 ? 0 : row / (32);
      if (i0 + prow < n)
        *reinterpret_cast<u32x4*>(obase + prow * orow_stride + hd * D + (tid % G::PPR) * 8) =
            *reinterpret_cast<const u32x4*>(lds + row * G::OS + (tid % G::PPR) * 8);
    }
  }
}

template <int D, int HW>
hipError_t run(const ltea_cfg& cfg, const void* q, int64_t q_st, int64_t q_sh, const void* k, const void* v,
               int64_t kv_st, int64_t kv_sh, const SeqView& sv, const ltea_cache& c, void* out,
               const int32_t* kv_start, const int32_t* kv_len, float* lse, hipStream_t stream) {
  constexpr int BMQ = Geo<D>::BM / HW;
  const float scale = cfg.softmax_scale > 0.f ? cfg.softmax_scale : 1.0f / sqrtf((float)cfg.D);
  const int64_t tiles_upper = (sv.total_tokens + BMQ - 1) / BMQ + sv.n_seqs;
  const int64_t n_work = tiles_upper * (cfg.Hq / HW);
  const int64_t grid = (n_work + 7) / 8 * 8;
  hipLaunchKernelGGL((attention_mfma_kernel<D, HW>), dim3((unsigned)grid), dim3(kThreads), 0, stream,
                     static_cast<const bf16_t*>(q), q_st, q_sh, static_cast<const bf16_t*>(k),
                     static_cast<const bf16_t*>(v), kv_st, kv_sh, sv.cu_seqlens, sv.n_seqs, (int)tiles_upper,
                     (int)n_work, cfg.Hq, cfg.Hkv, cfg.window, cfg.budget, scale * 1.4426950408889634f,
                     static_cast<const bf16_t*>(c.k_ret), static_cast<const bf16_t*>(c.v_ret), c.ret_pos, c.ret_count,
                     static_cast<bf16_t*>(out), kv_start, kv_len, lse, sv.total_tokens);
  return hipGetLastError();
}

}  // namespace

// The kernel addresses K/V rows of one sequence with 32-bit byte offsets.
bool attention_mfma_supported(const ltea_cfg& cfg, int64_t kv_stride_tok, int32_t max_seqlen) {
  if (cfg.dtype != LTEA_BF16 || (cfg.D != 64 && cfg.D != 128)) return false;
  return (int64_t)max_seqlen * kv_stride_tok * 2 < ((int64_t)1 << 31) && (int64_t)cfg.budget * cfg.D * 2 < ((int64_t)1 << 31);
}

hipError_t launch_attention_mfma(const ltea_cfg& cfg, const void* q, int64_t q_st, int64_t q_sh, const void* k,
                                 const void* v, int64_t kv_st, int64_t kv_sh, const SeqView& sv, const ltea_cache& c,
                                 void* out, hipStream_t stream, const int32_t* kv_start, const int32_t* kv_len,
                                 float* lse) {
  if (sv.total_tokens == 0) return hipSuccess;
  // grouped-query shapes with a multiple of four query heads per KV head: one query head per wave (see the kernel)
  const bool by_head = (cfg.Hq / cfg.Hkv) % 4 == 0;
  if (cfg.D == 64)
    return by_head ? run<64, 4>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, kv_start, kv_len, lse, stream)
                   : run<64, 1>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, kv_start, kv_len, lse, stream);
  return by_head ? run<128, 4>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, kv_start, kv_len, lse, stream)
                 : run<128, 1>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, kv_start, kv_len, lse, stream);
}

}  // namespace ltea
