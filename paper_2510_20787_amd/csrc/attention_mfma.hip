// Prefill attention over window + retained set (paper Section 3.1.3) on bf16 MFMA for gfx950.
//
// Flash-attention-style tiling, two stages per query tile as in the paper's description: stage 1 walks
// 64-key tiles of the original K/V inside the tile's window range, stage 2 walks 64-slot tiles of the
// compact retained segment with a per-row mask "position <= i - window" (so entries still inside a
// query's window are never counted twice).  Per wave, tiles wholly outside its rows' reach are skipped and
// only tiles that straddle a window edge, the causal diagonal, the sequence end or the visibility frontier of
// the retained entries pay for masking.
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
// K/V tiles are double-buffered in LDS and come there straight from global memory, one tile ahead, one barrier per tile
// (three workgroups share a CU at D = 64, two at D = 128; a 128-VGPR build of the D = 64 kernel reaches four but
// spills, which costs HBM traffic and gains no time).  There is no running maximum: a row's exponentials are taken
// relative to the maximum of the first block in which it sees a key (the result does not depend on that reference
// value as long as the exponentials stay in range; a workgroup whose row sums leave the range repeats its tiles with
// the exact running maximum), which keeps the row-maximum reduction and the accumulator rescale off the common path.
// What bounds it: the instruction stream of a wave, which issues in order.  A tile that every row of the wave sees whole takes
// a body without branches in which each matrix instruction of one 32-key block is followed by its share of the other block's
// exponentials.  Through registers and with a mask mode per block 32768 tokens x 32 heads (D = 128) took 1979 us, this form
// with the accumulators in place across the tile 1675 us; 4 x 4096 tokens, 16 heads of D = 64: 114 -> 105 us (whole prefill).
#include <type_traits>

#include "ltea_common.h"
#include "ltea_kernels.h"
#include "mfma_tiles.h"
#include "score_dma.h"

namespace ltea {
namespace {

constexpr int BN = 64;   // keys per tile
constexpr int kThreads = 256;
constexpr float kBig = 1.8446744e19f;  // 2^64: a row sum above this (or not a number) sends the workgroup through its tiles again

template <int D, int QB> struct Geo {
  static constexpr int BM = 128 * QB;           // queries per workgroup
  static constexpr int PPR = D / 8;             // 16-byte pieces per row
  static constexpr int RPI = 64 / PPR;          // rows per wave load instruction
  static constexpr int IPW = BN / RPI / 4;      // load instructions per wave, K tile and V tile each
  static constexpr int OS = D + 8;              // epilogue staging row stride (elements)
  static constexpr int kTile = BN * D;          // elements of one tile; K tile then V tile per buffer, rows unpadded
  static constexpr int kBuf = 2 * kTile;
};

// Which 16-byte piece of its row a K tile row keeps at slot p (p ^ term): the row reads of 16 consecutive lanes (16 rows at
// one piece) then cover all 64 banks.
template <int D> __device__ __forceinline__ int piece_swizzle(int row) { return D == 64 ? ((row >> 1) & 7) : (row & 15); }

// HW = query heads per workgroup.  1: the four waves take four consecutive blocks of 32 query positions of one head.
// 4 (grouped-query shapes with a multiple of four query heads per KV head): the four waves take the SAME 32 positions
// of four query heads that share the KV head.  The K/V tiles are shared either way, but with HW = 4 every wave sees the
// same window, so a tile is plain, masked or out of reach for all four at once (with HW = 1 the waves' windows are
// shifted by 32 positions each, the workgroup's key range is 96 positions longer, and whenever one wave has a masked
// tile the other three wait for it at the tile barrier).
template <int D, int QB, int HW>
__global__ void __launch_bounds__(kThreads, D == 64 ? 3 : 2)
attention_mfma_kernel(const bf16_t* __restrict__ q, int64_t q_st, int64_t q_sh, const bf16_t* __restrict__ k,
                      const bf16_t* __restrict__ v, int64_t kv_st, int64_t kv_sh, const int32_t* __restrict__ cu,
                      int n_seqs, int tiles_upper, int n_work, int Hq, int Hkv, int window, int budget,
                      float scale_log2e, const bf16_t* __restrict__ k_ret, const bf16_t* __restrict__ v_ret,
                      const int32_t* __restrict__ ret_pos, const int32_t* __restrict__ ret_count,
                      bf16_t* __restrict__ out, const int32_t* __restrict__ kv_start,
                      const int32_t* __restrict__ kv_len, float* __restrict__ lse, int64_t lse_stride) {
  using G = Geo<D, QB>;
  constexpr int BM = G::BM, kBuf = G::kBuf, kTile = G::kTile;
  constexpr int BMQ = BM / HW;     // query positions per workgroup (BM = rows of all its waves)
  static_assert(HW == 1 || HW == 4, "one head, or one head per wave");
  static_assert(2 * kBuf >= BM * G::OS, "epilogue staging must fit in the tile buffers");
  __shared__ __align__(1024) bf16_t lds[2 * kBuf];
  __shared__ __align__(256) int pos_lds[2][BN];
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
  const int r0 = i0 + (HW == 1 ? 32 * QB * wv : 0);               // first query row of this wave
  const int r_hi = r0 + 32 * QB - 1;        // last query row of this wave

  // ---- Q fragments (B operand of S^T): lane holds Q[row][16*ks + 8*hb .. +7] for its QB rows ------------
  bf16x8 qreg[QB][D / 16];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const int qi = r0 + 32 * qb + ql;
    const int qc = qi < n ? qi : n - 1;
    const bf16_t* qrow = q + (int64_t)(lo_q + qc - q_begin) * q_st + (int64_t)hq * q_sh;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) qreg[qb][ks] = *reinterpret_cast<const bf16x8*>(qrow + 16 * ks + 8 * hb);
  }

  // ---- tile schedule ------------------------------------------------------------------------------------
  const int i_last = (i0 + BMQ < n ? i0 + BMQ : n) - 1;          // last real query row of the workgroup
  const int jlo = i0 - window + 1 > 0 ? i0 - window + 1 : 0;
  const int jt0 = (jlo / BN) * BN;
  const int n_win_tiles = (i_last - jt0) / BN + 1;
  const int cnt = (budget > 0 && i_last - window >= 0) ? ret_count[head] : 0;
  const int n_ret_tiles = (cnt + BN - 1) / BN;
  const int n_tiles = n_win_tiles + n_ret_tiles;

  // ---- per-thread load addressing: buffer loads with 32-bit byte offsets; rows past the end of the sequence
  // (or past ret_count in the compact segment) are out of the descriptor's range and read as zeros ----------
  const uint32_t row_bytes = (uint32_t)kv_st * 2u;
  const uint32_t win_bytes = (uint32_t)(n - 1) * row_bytes + (uint32_t)(D * 2);
  const uint32_t ret_bytes = (uint32_t)cnt * (uint32_t)(D * 2);
  const u32x4 rs_k = make_raw_rsrc(k + lo * kv_st + (int64_t)h * kv_sh, win_bytes);
  const u32x4 rs_v = make_raw_rsrc(v + lo * kv_st + (int64_t)h * kv_sh, win_bytes);
  const u32x4 rs_kr = make_raw_rsrc(k_ret + head * budget * D, ret_bytes);
  const u32x4 rs_vr = make_raw_rsrc(v_ret + head * budget * D, ret_bytes);
  const u32x4 rs_pos = make_raw_rsrc(ret_pos + head * budget, (uint32_t)cnt * 4u);

  // ---- global -> LDS: a wave instruction fills RPI rows (1 KB) of one tile; instruction wv + 4*i.  The tiles are swizzled
  // by which piece a lane fetches: K for the row reads, V (its 64-byte chunks) for the transposing reads.  The swizzle terms
  // of a lane's rows do not depend on i.
  const int ld_row = G::RPI * wv + lane / G::PPR, ld_slot = lane % G::PPR;       // + 4 * RPI * i
  const uint32_t ld_k = (uint32_t)(ld_slot ^ piece_swizzle<D>(ld_row)) * 16u;
  const uint32_t ld_v = (uint32_t)((((ld_slot >> 2) ^ chunk_swizzle<D>(ld_row)) << 2) | (ld_slot & 3)) * 16u;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  const uint32_t pos_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&pos_lds[0][0];
  auto load_tile = [&](int t) {
    const bool win = t < n_win_tiles;
    const int row0 = win ? jt0 + t * BN : (t - n_win_tiles) * BN;
    const uint32_t rb = win ? row_bytes : (uint32_t)(D * 2);
    const uint32_t dst = lds_base + (uint32_t)((t & 1) * kBuf * 2 + wv * 1024);
    const u32x4 rk = win ? rs_k : rs_kr, rv = win ? rs_v : rs_vr;
    uint32_t row_off = (uint32_t)(row0 + ld_row) * rb;
#pragma unroll
    for (int i = 0; i < G::IPW; ++i) {
      dma16(rk, dst + (uint32_t)(i * 4096), row_off + ld_k);
      dma16(rv, dst + (uint32_t)(kTile * 2 + i * 4096), row_off + ld_v);
      row_off += (uint32_t)(4 * G::RPI) * rb;
    }
    if (!win && wv == 0)          // the tile's 64 positions (zeros past ret_count)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                   :: "s"(pos_base + (uint32_t)((t & 1) * BN * 4)), "v"((uint32_t)(row0 + lane) * 4u), "s"(rs_pos) : "memory");
  };

  // operand load offsets inside a tile buffer (elements).  K: MFMA row ql carries tile row kr; its pieces 2*ks + hb.
  const int k_row = tile_row_of_mfma_row(ql);
  const int k_off0 = k_row * D + ((piece_swizzle<D>(k_row) ^ hb) << 3);         // ^ (16 * ks), + 32 * D * kb
  // V operand through the transposing LDS load: in each group of 16 lanes, lane j points at the four columns
  // d0 + 4*(j%4).. of key row kbase + j/4, and receives column d0 + j of the four keys kbase..kbase+3.
  const int tr_key = 8 * hb + ((lane & 15) >> 2);           // + 32*kb + 16*kk (+ 4 for the upper half)
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);  // + 32*db, inside one 64-byte chunk
  const int tr_swz = chunk_swizzle<D>(tr_key);                  // unchanged by adding multiples of 4 to the key
  const int a_v_off = kTile + tr_key * D + tr_col;

  // ---- softmax state (per lane = per query; the two lane halves keep separate partial sums) ------
  float m_run[QB], l_part[QB];
  bool all_have_m = false;     // wave-uniform: every row of the wave has a reference value (m_run finite)
  bool exact_pass = false;     // workgroup-uniform: second run over the tiles, with the running maximum in every block
  f32x16 o[QB][D / 32];
  auto reset_rows = [&]() {
    all_have_m = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      m_run[qb] = -INFINITY;
      l_part[qb] = 0.f;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[qb][db][r] = 0.f;
    }
  };
  reset_rows();

  // mode: 0 = plain, 1 = window-edge mask (keys jt..), 2 = retained mask (positions in pos_lds).
  // The 64-key tile is consumed as two 32-key halves, each with its own softmax update, so that only one
  // 32x32 score block per query block is live at a time.
  // `slots`: entries of a retained tile.
  auto compute = [&](const int mode, const bf16_t* buf, const int* pos, int jt, int slots) {
    const bf16_t* a_v = buf + a_v_off;
    auto load_k_ops = [&](int kb, bf16x8 (&a)[D / 16]) {
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) a[ks] = *reinterpret_cast<const bf16x8*>(buf + (k_off0 ^ (16 * ks)) + 32 * D * kb);
    };
    auto score_block = [&](const bf16x8 (&a)[D / 16], f32x16 (&sc)[QB]) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[qb][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
          sc[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], qreg[qb][ks], sc[qb], 0, 0, 0);
    };
    // mask: register r is local key 32*kb + 16*(r/8) + 8*hb + r%8
    auto apply_mask = [&](int kb, f32x16 (&scs)[QB]) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        f32x16& sc = scs[qb];
        const int qi = r0 + 32 * qb + ql;
        if (mode == 1) {
          // valid local keys c (without the 8*hb term) form the range [c_lo, c_hi]: causal, window and sequence end
          const int shift = jt + 8 * hb;
          int c_hi = qi - shift;                                   // j <= qi
          const int c_end = n - 1 - shift;                         // j <= n-1
          c_hi = c_hi < c_end ? c_hi : c_end;
          int c_lo = qi - window + 1 - shift;                      // j >= qi - window + 1
          const unsigned span = c_hi >= c_lo ? (unsigned)(c_hi - c_lo) : 0u;
          if (c_hi < c_lo) c_lo = 0x40000000;                      // nothing valid
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int c = 32 * kb + 16 * (r / 8) + (r % 8);
            sc[r] = ((unsigned)(c - c_lo) <= span) ? sc[r] : -INFINITY;
          }
        } else if (mode == 2) {
          const int lim = qi - window;
#pragma unroll
          for (int r8 = 0; r8 < 2; ++r8) {
            const int* pp = pos + 32 * kb + 16 * r8 + 8 * hb;
#pragma unroll
            for (int e = 0; e < 8; ++e) sc[8 * r8 + e] = (pp[e] <= lim && 32 * kb + 16 * r8 + 8 * hb + e < slots) ? sc[8 * r8 + e] : -INFINITY;
          }
        }
      }
    };
    // The reference value m of a row (probabilities are exp2(score - m)) only has to keep the exponentials in range,
    // so it is not the running maximum: a row takes the maximum of the first block in which it sees a key and keeps it
    // (l is then at least the 1 of that block, and the softmax is the same function of the scores for any m).  Scores
    // that later exceed m by more than the exponent range allows show up as a huge or non-finite row sum when the
    // tiles are done; the workgroup then runs its tiles a second time with the exact running maximum in every block.
    auto raise_reference = [&](const f32x16 (&scs)[QB]) {
      bool still_none = false;
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const f32x16& sc = scs[qb];
        float mx = fmaxf(sc[0], sc[1]);
#pragma unroll
        for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, sc[r]), sc[r + 1]);
        mx = pair_max(mx);
        const float m_new = fmaxf(m_run[qb], mx * scale_log2e);
        // nothing visible so far and nothing now: m stays -inf, and the factor must not become exp2(nan)
        const float a = (m_new == m_run[qb]) ? 1.0f : __builtin_amdgcn_exp2f(m_run[qb] - m_new);
        m_run[qb] = m_new;
        l_part[qb] *= a;
        if (__builtin_amdgcn_ballot_w64(a != 1.0f) != 0ull) {
#pragma unroll
          for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[qb][db][r] *= a;
        }
        still_none = still_none || (m_new == -INFINITY);
      }
      all_have_m = __builtin_amdgcn_ballot_w64(still_none) == 0ull;
    };
    auto exp_block = [&](const f32x16 (&scs)[QB], bf16x8 (&pb)[QB][2], float (&psum)[QB]) {
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const float m_use = (m_run[qb] == -INFINITY) ? 0.f : m_run[qb];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(fmaf(scs[qb][r], scale_log2e, -m_use));
          pb[qb][r / 8][r % 8] = static_cast<bf16_t>(p);
        }
        // Row sum from the rounded probabilities, two per instruction (v_dot2c_f32_bf16 with a vector of ones):
        // the denominator then matches the bf16 P that the second MFMA consumes.
        bf16x2 ones;
        ones[0] = static_cast<bf16_t>(1.0f); ones[1] = static_cast<bf16_t>(1.0f);
        float psum0 = 0.f, psum1 = 0.f;
#pragma unroll
        for (int r2 = 0; r2 < 8; r2 += 2) {
          bf16x2 e0, e1;
          e0[0] = pb[qb][r2 / 4][(2 * r2) % 8]; e0[1] = pb[qb][r2 / 4][(2 * r2) % 8 + 1];
          e1[0] = pb[qb][r2 / 4][(2 * r2) % 8 + 2]; e1[1] = pb[qb][r2 / 4][(2 * r2) % 8 + 3];
          psum0 = __builtin_amdgcn_fdot2_f32_bf16(e0, ones, psum0, false);
          psum1 = __builtin_amdgcn_fdot2_f32_bf16(e1, ones, psum1, false);
        }
        psum[qb] = psum0 + psum1;
      }
    };
    // Softmax of one 32-key block whose (masked) scores are in s: probabilities to p, row sums to l_part
    auto softmax_block = [&](int kb, f32x16 (&s)[QB], bf16x8 (&p)[QB][2]) {
      float psum[QB];
      if (!all_have_m || exact_pass) raise_reference(s);
      exp_block(s, p, psum);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        l_part[qb] += psum[qb];
        // Pin the packed probabilities here: without a use in this block the compiler sinks the exponentials
        // past the following branches, away from the MFMAs they are meant to overlap with.
        u32x4 w0 = __builtin_bit_cast(u32x4, p[qb][0]), w1 = __builtin_bit_cast(u32x4, p[qb][1]);
        asm volatile("" : "+v"(w0), "+v"(w1), "+v"(l_part[qb]));
        p[qb][0] = __builtin_bit_cast(bf16x8, w0);
        p[qb][1] = __builtin_bit_cast(bf16x8, w1);
      }
    };
    auto load_v_ops = [&](int kb, bf16x8 (&av)[D / 32][2]) {
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        const bf16_t* ap = a_v + 32 * kb * D + ((db ^ tr_swz) << 5);
        av[db][0] = load_transposed(ap, D);
        av[db][1] = load_transposed(ap + 16 * D, D);
      }
    };
    auto pv_block = [&](const bf16x8 (&av)[D / 32][2], const bf16x8 (&pb)[QB][2]) {   // O^T += V^T P^T
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          o[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[db][0], pb[qb][0], o[qb][db], 0, 0, 0);
          o[qb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[db][1], pb[qb][1], o[qb][db], 0, 0, 0);
        }
    };
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      f32x16 s[QB];
      bf16x8 p[QB][2], ak[D / 16], av[D / 32][2];
      load_k_ops(kb, ak);
      score_block(ak, s);
      apply_mask(kb, s);
      softmax_block(kb, s, p);
      load_v_ops(kb, av);
      pv_block(av, p);
    }
  };

  // A tile that every row of the wave sees whole, once all rows have a reference value: the same products and exponentials
  // without a branch in between, so that the instruction stream can interleave them.  A wave issues in order and a matrix
  // instruction occupies the matrix pipe for 32 clocks after its issue: vector instructions placed behind it run in that
  // time, those behind the last one of a row of matrix instructions do not.
  auto compute_plain = [&](const bf16_t* buf) {
    constexpr int NK = D / 16, ND = D / 32;
    const bf16_t* a_v = buf + a_v_off;
    auto k_op = [&](int kb, int ks) { return *reinterpret_cast<const bf16x8*>(buf + (k_off0 ^ (16 * ks)) + 32 * D * kb); };
    auto v_op = [&](int kb, int db, int kk) { return load_transposed(a_v + 32 * kb * D + ((db ^ tr_swz) << 5) + 16 * kk * D, D); };
    auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
    bf16x2 ones;
    ones[0] = static_cast<bf16_t>(1.0f); ones[1] = static_cast<bf16_t>(1.0f);
    // softmax of elements EPM*i .. of a block, behind its i-th matrix instruction: exponentials now, conversion and row sum
    // of the elements of the step before
    constexpr int EPM = 16 / NK;
    float e[16], l0 = 0.f, l1 = 0.f;
    auto exp_part = [&](int i, const f32x16& sc) {
#pragma unroll
      for (int r = EPM * i; r < EPM * (i + 1); ++r) {
        e[r] = __builtin_amdgcn_exp2f(fmaf(sc[r], scale_log2e, -m_run[0]));
        asm volatile("" : "+v"(e[r]));      // here, not next to its first use
      }
    };
    auto pin = [](bf16x8& x) {
      u32x4 w = __builtin_bit_cast(u32x4, x);
      asm volatile("" : "+v"(w));
      x = __builtin_bit_cast(bf16x8, w);
    };
    auto pack_part = [&](int i, bf16x8 (&p)[2]) {
#pragma unroll
      for (int r = EPM * i; r < EPM * (i + 1); r += 2) {
        bf16x2 x;
        x[0] = static_cast<bf16_t>(e[r]); x[1] = static_cast<bf16_t>(e[r + 1]);
        p[r / 8][r % 8] = x[0]; p[r / 8][r % 8 + 1] = x[1];
        if (r % 4 == 0) l0 = __builtin_amdgcn_fdot2_f32_bf16(x, ones, l0, false);
        else l1 = __builtin_amdgcn_fdot2_f32_bf16(x, ones, l1, false);
      }
    };
    f32x16 s0, s1;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s0[r] = 0.f; s1[r] = 0.f; }
    bf16x8 p0[2], p1[2], ka[NK], kb[NK], va[NK], vb[NK];     // value operands in the order (kk, db)
#pragma unroll
    for (int i = 0; i < NK; ++i) ka[i] = k_op(0, i);
    fence();
#pragma unroll
    for (int i = 0; i < NK; ++i) {                       // scores of block 0, reading block 1's keys
      pin(ka[i]);
      s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i], qreg[0][i], s0, 0, 0, 0);
      kb[i] = k_op(1, i);
      fence();
    }
#pragma unroll
    for (int i = 0; i < NK; ++i) {                       // scores of block 1 / softmax of block 0 / values of block 0
      pin(kb[i]);
      s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[i], qreg[0][i], s1, 0, 0, 0);
      va[i] = v_op(0, i % ND, i / ND);
      exp_part(i, s0);
      if (i > 0) pack_part(i - 1, p0);
      fence();
    }
    pack_part(NK - 1, p0);
    fence();
#pragma unroll
    for (int i = 0; i < NK; ++i) {                       // value products of block 0 / softmax of block 1 / values of block 1
      pin(va[i]);
      o[0][i % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i], p0[i / ND], o[0][i % ND], 0, 0, 0);
      vb[i] = v_op(1, i % ND, i / ND);
      exp_part(i, s1);
      if (i > 0) pack_part(i - 1, p1);
      fence();
    }
    pack_part(NK - 1, p1);
    l_part[0] += l0 + l1;
    fence();
#pragma unroll
    for (int i = 0; i < NK; ++i)
      o[0][i % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb[i], p1[i / ND], o[0][i % ND], 0, 0, 0);
    fence();
  };

  // ---- tile t is computed from LDS buffer t&1 while tile t+1 is on its way into the other one ---------------------
  auto step = [&](int t) {
    if (t + 1 < n_tiles) load_tile(t + 1);      // everyone is done with tile t-1, whose buffer this is
    const bf16_t* buf = lds + (t & 1) * kBuf;
    // classify the tile for this wave: -1 skip, 0 every (query, key) pair valid, 1 window-edge mask, 2 retained mask
    int mode = -1, jt = 0, slots = 0;
    if (r0 < n) {
      if (t < n_win_tiles) {
        jt = jt0 + t * BN;
        // keys this wave can use at all: [r0 - window + 1, r_hi]
        if (!(jt > r_hi || jt + BN - 1 < r0 - window + 1))
          mode = ((jt + BN - 1 <= r0) && (jt >= r_hi - window + 1)) ? 0 : 1;
      } else {
        // every wave looks at the tile's positions itself (one LDS word per lane, two compares): an entry counts for
        // this wave once it has left the window of the wave's last row, and needs no mask once it has left the window
        // of the first; the slots past the last entry never do
        slots = cnt - (t - n_win_tiles) * BN;
        int pv = pos_lds[t & 1][lane];
        pv = lane < slots ? pv : 0x7FFFFFFF;
        if (__builtin_amdgcn_ballot_w64(pv <= r_hi - window) != 0ull)
          mode = __builtin_amdgcn_ballot_w64(pv > r0 - window) == 0ull ? 0 : 2;
      }
    }
    mode = __builtin_amdgcn_readfirstlane(mode);
    // Two steps in sequence rather than if / else: as an alternative of the plain body the other one kept the accumulators of
    // before the tile alive across it, and every tile ended with waiting for its last products and copying them.
    if (mode == 0 && all_have_m && !exact_pass) {
      compute_plain(buf);
      mode = -1;
    }
    asm volatile("" : "+s"(mode));
    if (mode >= 0) compute(mode, buf, pos_lds[t & 1], jt, slots);
    wait_loads();
    __syncthreads();   // tile t+1 is in LDS; everyone is done with tile t
  };
  if (tid == 0) redo_flag = 0;
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    load_tile(0);
    wait_loads();
    __syncthreads();
#pragma unroll 1
    for (int t = 0; t < n_tiles; ++t) step(t);
    if (exact_pass) break;
    // did a row's reference value fall so far below its scores that its sums left the range?
    bool bad = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) bad = bad || !(l_part[qb] <= kBig);
    if (__builtin_amdgcn_ballot_w64(bad) != 0ull && lane == 0) redo_flag = 1;
    __syncthreads();  // also: tile buffers are free
    if (__builtin_amdgcn_readfirstlane(redo_flag) == 0) break;
    exact_pass = true;
    reset_rows();
  }

  // ---- epilogue: normalise, stage through LDS, store rows coalesced -------------------------------------------
  __syncthreads();  // tile buffers are free
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float l_row = pair_sum(l_part[qb]);
    const float inv = 1.0f / l_row;
    if (lse != nullptr && hb == 0) {
      // natural-log normaliser of the scaled scores (m_run is kept in the base-2 domain); wanted by a backward pass
      const int row = (HW == 1 ? 32 * QB * wv : 0) + 32 * qb + ql;
      if (i0 + row < n) lse[(int64_t)hq * lse_stride + lo_q + i0 + row - q_begin] = (m_run[qb] + __log2f(l_row)) * 0.6931471805599453f;
    }
    bf16_t* orow = lds + (32 * QB * wv + 32 * qb + ql) * G::OS + 4 * hb;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        bf16x4 w4;
#pragma unroll
        for (int e = 0; e < 4; ++e) w4[e] = static_cast<bf16_t>(o[qb][db][4 * g4 + e] * inv);
        *reinterpret_cast<bf16x4*>(orow + 32 * db + 8 * g4) = w4;
      }
  }
  __syncthreads();
  {
    // staging row = 32*QB*wave + position block: with HW = 1 all rows are positions of one head, with HW = 4 the
    // wave index is the head inside the group
    bf16_t* obase = out + ((int64_t)(lo_q + i0 - q_begin) * Hq + unit * HW) * D;
    const int64_t orow_stride = (int64_t)Hq * D;
    constexpr int kRowsPerPass = kThreads / G::PPR;
#pragma unroll
    for (int p = 0; p < BM / kRowsPerPass; ++p) {
      const int row = p * kRowsPerPass + tid / G::PPR;
      const int prow = HW == 1 ? row : row % (32 * QB), hd = HW == 1 ? 0 : row / (32 * QB);
      if (i0 + prow < n)
        *reinterpret_cast<u32x4*>(obase + prow * orow_stride + hd * D + (tid % G::PPR) * 8) =
            *reinterpret_cast<const u32x4*>(lds + row * G::OS + (tid % G::PPR) * 8);
    }
  }
}

template <int D, int QB, int HW>
hipError_t run(const ltea_cfg& cfg, const void* q, int64_t q_st, int64_t q_sh, const void* k, const void* v,
               int64_t kv_st, int64_t kv_sh, const SeqView& sv, const ltea_cache& c, void* out,
               const int32_t* kv_start, const int32_t* kv_len, float* lse, hipStream_t stream) {
  constexpr int BMQ = Geo<D, QB>::BM / HW;
  const float scale = cfg.softmax_scale > 0.f ? cfg.softmax_scale : 1.0f / sqrtf((float)cfg.D);
  const int64_t tiles_upper = (sv.total_tokens + BMQ - 1) / BMQ + sv.n_seqs;
  const int64_t n_work = tiles_upper * (cfg.Hq / HW);
  const int64_t grid = (n_work + 7) / 8 * 8;
  hipLaunchKernelGGL((attention_mfma_kernel<D, QB, HW>), dim3((unsigned)grid), dim3(kThreads), 0, stream,
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
    return by_head ? run<64, 1, 4>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, kv_start, kv_len, lse, stream)
                   : run<64, 1, 1>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, kv_start, kv_len, lse, stream);
  return by_head ? run<128, 1, 4>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, kv_start, kv_len, lse, stream)
                 : run<128, 1, 1>(cfg, q, q_st, q_sh, k, v, kv_st, kv_sh, sv, c, out, kv_start, kv_len, lse, stream);
}

}  // namespace ltea
