// Training-side backward of the SWA+LTE attention on bf16 MFMA for gfx950, head dimensions 64 and 128 (paper
// Section 3.1.2: the gradients that reach Q, K, V and, through the straight-through estimator, the retention scores).
//
// Three launches on the caller's stream:
//   train_delta_mfma_kernel      delta = <dO, O> and lse, scaled, per (query, query head).
//   train_dq_far_mfma_kernel     two independent roles in one grid: the far pass of dK / dV (first, few and
//                                long-running workgroups) and dQ (fills the compute units the far pass leaves idle).
//   train_dkv_band_mfma_kernel   the band pass of dK / dV, which adds the far pass in, stores dK, dV and forms
//                                d logit and the retention counts.
//
// dQ role: one workgroup = 128 consecutive queries of one (sequence, query head), 4 waves x 32 queries (or 32 queries of four
// heads, one per wave, see dq_body), walking 64-key tiles of K/V on a fixed grid inside the window range, then 64-slot tiles of
// the compacted candidates with the per-row mask "position <= i - window" (the forward kernel has since gone over to blocks of
// 32 keys aligned to the query rows, with masked tiles interleaved like plain ones; this one has not).  Per 32-key block
// and wave (v_mfma_f32_32x32x16_bf16, a lane owns one query column):
//   S^T[key, query]  = K . Q^T        A = K tile rows from LDS, B = Q fragment in registers
//   dP^T[key, query] = V . dO^T       A = V tile rows from LDS, B = dO fragment in registers
//   P^T = exp2((S^T - lse / scale) c), dS^T = P^T (dP^T - delta)      no running maximum
//   dQ^T[d, query]  += K^T . dS^T     A = K^T through the transposing LDS load, B = dS^T straight from registers
// The two differences cost nothing: the products' accumulators start from -lse / scale and -delta.  The exponent then carries
// the rounding of sums of that size instead of one multiply-add's; against 64 bits nothing of it is left beside P and dS in
// bf16: relative error of dQ, dK, dV at 1300 tokens of the paper's layer 2.4893e-3, 2.4564e-3, 2.3300e-3 with the
// subtractions behind the products, 2.4893e-3, 2.4562e-3, 2.3300e-3 in this form, and with queries 16 times as large (lse to
// 102) 6.250e-3, 5.887e-3, 2.340e-3 and 6.249e-3, 5.886e-3, 2.339e-3.
// The dK / dV roles are the mirror image with a lane owning a key column (see dkv_body).
// What bounds them: the instruction stream of a wave, which issues in order.  Tiles come straight into LDS, one copy each,
// swizzled so that the row reads and the transposing reads of it are both free of bank conflicts; a tile that every row of the
// wave sees whole takes a body without branches in which each matrix instruction is followed by its share of the exponentials
// (4.3 VALU per matrix instruction in dK / dV, 5 in dQ, from 10 to 12 when tiles went through registers, K / Q / dO were
// stored twice and every block was a basic block of its own).  4 x 4096 tokens, 32 heads on 8, D = 64, window 768, an eighth
// kept: dQ with the far pass 467 -> 363 us (378 with consecutive blocks of one head on the waves), band pass 359 -> 285 us.
// Candidates that no row of a dQ workgroup sees (half of them on average, all of them later positions) are neither loaded nor
// waited for, and a masked tile leaves out a block of 32 that nobody of the wave sees (in either role): the whole training
// step of that layer 1026 -> 1012 us, both forms in turn on one box, with the same results.
// Two tile buffers, one barrier per tile.  No floating-point atomics: the partial sums of the far pass go to scratch slices
// that the band pass adds in a fixed order.
#include <type_traits>

#include "ltea_common.h"
#include "ltea_kernels.h"
#include "mfma_tiles.h"
#include "score_dma.h"
#include "train_common.h"

namespace ltea {
namespace {

constexpr int BN = 64;          // keys (or queries) per tile
constexpr int BM = 128;         // queries (or keys) per workgroup
constexpr int kThreads = 256;
constexpr int kStage = 2;       // tiles between two barriers

template <int D> struct Geo {
  static constexpr int PPR = D / 8;             // 16-byte pieces per row
  static constexpr int RPP = kThreads / PPR;    // rows per epilogue pass
  static constexpr int RPI = 64 / PPR;          // rows per wave load instruction
  static constexpr int IPW = BN / RPI / 4;      // load instructions per wave, each of the two tiles of a step
  static constexpr int OS = D + 8;              // epilogue staging stride
  static constexpr int kTile = BN * D;          // elements of one tile; a buffer holds two (K and V, or Q and dO)
  static constexpr int kBuf = 2 * kTile;
};
#define LTEA_GEO(D) \
  using G_ = Geo<D>; \
  constexpr int PPR = G_::PPR, RPP = G_::RPP, OS = G_::OS, kTile = G_::kTile, kBuf = G_::kBuf

// Where a lane finds its operands in a tile (see both_ways_swizzle): row reads (A operand = tile rows) and transposing
// reads (contraction over the tile rows) of the same copy.
template <int D> struct Operands {
  int row_off, tr_off;
  __device__ __forceinline__ explicit Operands(int lane) {
    const int ql = lane & 31, hb = lane >> 5;
    const int m_row = tile_row_of_mfma_row(ql);
    row_off = m_row * D + ((both_ways_swizzle<D>(m_row) ^ hb) << 3);
    const int tr_row = 8 * hb + ((lane & 15) >> 2);
    const int piece = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    tr_off = tr_row * D + ((both_ways_swizzle<D>(tr_row) ^ piece) << 3) + 4 * (lane & 1);
  }
  // tile rows 32 * blk .., features 16 * ks ..
  __device__ __forceinline__ bf16x8 rows(const bf16_t* t, int blk, int ks) const {
    return *reinterpret_cast<const bf16x8*>(t + (row_off ^ (16 * ks)) + 32 * D * blk);
  }
  // features 32 * db .., contraction over tile rows 32 * blk + 16 * kk ..
  __device__ __forceinline__ bf16x8 columns(const bf16_t* t, int blk, int kk, int db) const {
    const bf16_t* p = t + (32 * blk + 16 * kk) * D;
    return load_transposed_at(p + (tr_off ^ (32 * db)), p + 4 * D + (tr_off ^ 8 ^ (32 * db)));
  }
};

// f(0), f(1), .. f(N - 1) with the index as a constant (the compiler's own unrolling gives up on bodies of this size).
template <int N, int I = 0, class F> __device__ __forceinline__ void static_for(const F& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

__device__ __forceinline__ void pin(bf16x8& x) {
  u32x4 w = __builtin_bit_cast(u32x4, x);
  asm volatile("" : "+v"(w));
  x = __builtin_bit_cast(bf16x8, w);
}

// HW = query heads per workgroup.  1: the four waves take four consecutive blocks of 32 queries of one head.  4 (a multiple of
// four query heads per KV head): the same 32 queries of four heads that share the KV head, so that all four waves see the
// same window: the workgroup walks 96 positions less of it, and no wave waits at the barrier for another's masked tile.
template <int D, int HW>
__device__ __forceinline__ void dq_body(const TrainArgs& A, int tiles_upper, int n_work, float scale_log2e, int block,
                                        bf16_t* lds, int* pos_lds_base) {
  LTEA_GEO(D);
  static_assert(2 * kStage * kBuf >= BM * OS, "epilogue staging must fit in the tile buffers");

  const int per_xcd = (n_work + 7) / 8;
  const int work = (block % 8) * per_xcd + block / 8;
  if (work >= n_work) return;
  constexpr int BMQ = BM / HW;               // query positions per workgroup
  const int unit = work / tiles_upper;       // query head, or group of HW of them
  int tile, s, n, lo;
  if (!locate_tile(A.cu, A.n_seqs, BMQ, work - unit * tiles_upper, s, tile, lo, n)) return;
  const int Hq = A.Hq, Hkv = A.Hkv, window = A.window, budget = A.budget;
  const int h = unit * HW / (Hq / Hkv);
  const int64_t head = (int64_t)s * Hkv + h;
  const int i0 = tile * BMQ;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ql = lane & 31, hb = lane >> 5;
  const int hq = HW == 1 ? unit : unit * HW + wv;
  const int r0 = i0 + (HW == 1 ? 32 * wv : 0);
  const int r_hi = r0 + 31;

  const bf16_t* q = static_cast<const bf16_t*>(A.q);
  const bf16_t* k = static_cast<const bf16_t*>(A.k);
  const bf16_t* v = static_cast<const bf16_t*>(A.v);
  const bf16_t* dout = static_cast<const bf16_t*>(A.dout);

  // ---- per-lane query state: Q and dO fragments (B operands), -lse / scale and -delta --------------------------
  const int qi = r0 + ql;
  const int qc = qi < n ? qi : n - 1;
  bf16x8 qreg[D / 16], doreg[D / 16];
  {
    const bf16_t* qrow = q + (int64_t)(lo + qc) * A.q_st + (int64_t)hq * A.q_sh;
    const bf16_t* dorow = dout + ((int64_t)(lo + qc) * Hq + hq) * D;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      qreg[ks] = *reinterpret_cast<const bf16x8*>(qrow + 16 * ks + 8 * hb);
      doreg[ks] = *reinterpret_cast<const bf16x8*>(dorow + 16 * ks + 8 * hb);
    }
  }
  const int64_t stat = (int64_t)hq * A.total + lo + qc;
  const float neg_dlt = A.delta[stat], neg_lse = A.delta[(int64_t)Hq * A.total + stat];

  // ---- tile schedule: 64-key tiles from the multiple of 64 at or before the window's first key ------------------
  const int i_last = (i0 + BMQ < n ? i0 + BMQ : n) - 1;
  const int jlo = i0 - window + 1 > 0 ? i0 - window + 1 : 0;
  const int jt0 = (jlo / BN) * BN;
  const int n_win_tiles = (i_last - jt0) / BN + 1;
  const int cnt = (budget > 0 && i_last - window >= 0) ? A.ret_count[head] : 0;
  int n_tiles = n_win_tiles + (cnt + BN - 1) / BN;

  const uint32_t row_bytes = (uint32_t)A.kv_st * 2u;
  const uint32_t win_bytes = (uint32_t)(n - 1) * row_bytes + (uint32_t)(D * 2);
  const uint32_t ret_bytes = (uint32_t)cnt * (uint32_t)(D * 2);
  const u32x4 rs_k = make_raw_rsrc(k + (int64_t)lo * A.kv_st + (int64_t)h * A.kv_sh, win_bytes);
  const u32x4 rs_v = make_raw_rsrc(v + (int64_t)lo * A.kv_st + (int64_t)h * A.kv_sh, win_bytes);
  const u32x4 rs_kr = make_raw_rsrc(static_cast<const bf16_t*>(A.k_ret) + head * budget * D, ret_bytes);
  const u32x4 rs_vr = make_raw_rsrc(static_cast<const bf16_t*>(A.v_ret) + head * budget * D, ret_bytes);
  const u32x4 rs_pos = make_raw_rsrc(A.ret_pos + head * budget, (uint32_t)cnt * 4u);
  // global -> LDS: a wave instruction fills RPI rows (1 KB) of a tile, instruction wv + 4 * i; which piece a lane fetches
  // makes the swizzle, whose term does not depend on i
  const int ld_row = G_::RPI * wv + lane / PPR;
  const uint32_t ld_col = (uint32_t)((lane % PPR) ^ both_ways_swizzle<D>(ld_row)) * 16u;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  const uint32_t pos_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)pos_lds_base;
  auto load_tile = [&](int t) {
    const bool win = t < n_win_tiles;
    const int row0 = win ? jt0 + t * BN : (t - n_win_tiles) * BN;
    const uint32_t rb = win ? row_bytes : (uint32_t)(D * 2);
    const uint32_t dst = lds_base + (uint32_t)((t % (2 * kStage)) * kBuf * 2 + wv * 1024);
    const u32x4 rk = win ? rs_k : rs_kr, rv = win ? rs_v : rs_vr;
    uint32_t off = (uint32_t)(row0 + ld_row) * rb + ld_col;
#pragma unroll
    for (int i = 0; i < G_::IPW; ++i) {
      dma16(rk, dst + (uint32_t)(i * 4096), off);
      dma16(rv, dst + (uint32_t)(kTile * 2 + i * 4096), off);
      off += (uint32_t)(4 * G_::RPI) * rb;
    }
    if (!win && wv == 0) dma4(rs_pos, pos_base + (uint32_t)((t % (2 * kStage)) * BN * 4), (uint32_t)(row0 + lane) * 4u);   // zeros past cnt
  };
  const Operands<D> op(lane);
  constexpr int NK = D / 16, ND = D / 32;

  f32x16 acc[ND];
  f32x16 neg_lse16, neg_dlt16;       // the products start from these: S - lse / scale and dP - delta come out of the pipe
#pragma unroll
  for (int r = 0; r < 16; ++r) {
#pragma unroll
    for (int db = 0; db < ND; ++db) acc[db][r] = 0.f;
    neg_lse16[r] = neg_lse;
    neg_dlt16[r] = neg_dlt;
  }

  // mode: 1 = window-edge mask, 2 = mask by the candidates' positions (`slots`: entries of the tile); bit kb of `live`: some
  // row of the wave sees a key of block kb
  auto compute = [&](const int mode, const int live, const bf16_t* tb, const int* pos, int jt, int slots) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      if ((live >> kb & 1) == 0) continue;
      f32x16 sc = neg_lse16, dp = neg_dlt16;
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.rows(tb, kb, ks), qreg[ks], sc, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.rows(tb + kTile, kb, ks), doreg[ks], dp, 0, 0, 0);
      }
      // register r is local key 32*kb + 16*(r/8) + 8*hb + r%8
      if (mode == 1) {
        const int shift = jt + 8 * hb;
        int c_hi = qi - shift;
        const int c_end = n - 1 - shift;
        c_hi = c_hi < c_end ? c_hi : c_end;
        int c_lo = qi - window + 1 - shift;
        const unsigned span = c_hi >= c_lo ? (unsigned)(c_hi - c_lo) : 0u;
        if (c_hi < c_lo) c_lo = 0x40000000;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int c = 32 * kb + 16 * (r / 8) + (r % 8);
          sc[r] = ((unsigned)(c - c_lo) <= span) ? sc[r] : -INFINITY;
        }
      } else {
        const int lim = qi - window;
#pragma unroll
        for (int r8 = 0; r8 < 2; ++r8) {
          const int c0 = 32 * kb + 16 * r8 + 8 * hb;
#pragma unroll
          for (int e = 0; e < 8; ++e) sc[8 * r8 + e] = (pos[c0 + e] <= lim && c0 + e < slots) ? sc[8 * r8 + e] : -INFINITY;
        }
      }
      bf16x8 pb[2];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(sc[r] * scale_log2e);   // exp2(-inf) = 0 for masked pairs
        pb[r / 8][r % 8] = static_cast<bf16_t>(p * dp[r]);
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int db = 0; db < ND; ++db)
          acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.columns(tb, kb, kk, db), pb[kk], acc[db], 0, 0, 0);
    }
  };

  // A tile that every row of the wave sees whole: 6 NK matrix instructions without a branch, the exponentials of one block
  // behind the products of the other.  A wave issues in order and a matrix instruction holds the matrix pipe for 32 clocks
  // after its issue; vector instructions and LDS reads placed behind it run in that time.
  auto compute_plain = [&](const bf16_t* tb) {
    auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
    auto operand = [&](int i) {          // of the tile's i-th matrix instruction
      if (i < 4 * NK) return op.rows(tb + ((i & 1) ? kTile : 0), i / (2 * NK), (i % (2 * NK)) / 2);
      const int j = i - 4 * NK;
      return op.columns(tb, j / NK, (j % NK) / ND, j % ND);
    };
    constexpr int kAhead = 8;            // operands on their way from LDS
    bf16x8 x[kAhead], p0[2], p1[2];
    f32x16 s0 = neg_lse16, d0 = neg_dlt16, s1 = neg_lse16, d1 = neg_dlt16;
    float e[16];
    auto exps = [&](int i, int per, const f32x16& s, const f32x16& d) {
#pragma unroll
      for (int r = per * i; r < per * (i + 1); ++r) {
        e[r] = __builtin_amdgcn_exp2f(s[r] * scale_log2e) * d[r];
        asm volatile("" : "+v"(e[r]));      // here, not next to its first use
      }
    };
    auto pack = [&](int i, int per, bf16x8 (&p)[2]) {
#pragma unroll
      for (int r = per * i; r < per * (i + 1); ++r) p[r / 8][r % 8] = static_cast<bf16_t>(e[r]);
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) x[i] = operand(i);
    fence();
    static_for<6 * NK>([&](auto index) {
      constexpr int i = decltype(index)::value;
      bf16x8& a = x[i % kAhead];
      pin(a);
      constexpr int j = i % (2 * NK), ks = j / 2;
      if constexpr (i < 2 * NK) {                            // products of block 0
        if (j & 1) d0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, doreg[ks], d0, 0, 0, 0);
        else s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], s0, 0, 0, 0);
      } else if constexpr (i < 4 * NK) {                     // products of block 1 / exponentials of block 0
        if (j & 1) d1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, doreg[ks], d1, 0, 0, 0);
        else s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[ks], s1, 0, 0, 0);
      } else if constexpr (i < 5 * NK) {                     // dQ of block 0 / exponentials of block 1
        constexpr int m = i - 4 * NK;
        acc[m % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p0[m / ND], acc[m % ND], 0, 0, 0);
      } else {                                     // dQ of block 1
        constexpr int m = i - 5 * NK;
        acc[m % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p1[m / ND], acc[m % ND], 0, 0, 0);
      }
      if constexpr (i + kAhead < 6 * NK) a = operand(i + kAhead);
      if constexpr (i >= 2 * NK && i < 4 * NK) {
        constexpr int per = 8 / NK;
        constexpr int m = i - 2 * NK;
        exps(m, per, s0, d0);
        if (m > 0) pack(m - 1, per, p0);
        if (m == 2 * NK - 1) pack(m, per, p0);
      } else if constexpr (i >= 4 * NK && i < 5 * NK) {
        constexpr int per = 16 / NK;
        constexpr int m = i - 4 * NK;
        exps(m, per, s1, d1);
        if (m > 0) pack(m - 1, per, p1);
        if (m == NK - 1) pack(m, per, p1);
      }
      fence();
    });
  };

  // a stage of tiles is computed while the next one is on its way into the other half of the buffers
  auto load_stage = [&](int t0) {
#pragma unroll
    for (int t = t0; t < t0 + kStage; ++t)
      if (t < n_tiles) load_tile(t);
  };
  load_stage(0);
  // Under the flight of the first tiles: how many candidates have left the window of the last row (positions ascend, 64 of them
  // looked at per step).  The later ones are neither loaded nor waited for: half of them on average.
  {
    const int* rp = A.ret_pos + head * budget;
    const int lim = i_last - window;
    int seen = 0, left = cnt;
    while (left > 0) {
      const int step = (left + 63) / 64;
      const bool le = lane * step < left && rp[seen + lane * step] <= lim;
      const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(le));
      if (c == 0) break;
      const int end = seen + left;
      seen += (c - 1) * step + 1;
      left = step - 1 < end - seen ? step - 1 : end - seen;
    }
    n_tiles = n_win_tiles + (__builtin_amdgcn_readfirstlane(seen) + BN - 1) / BN;
  }
  wait_loads();
  __syncthreads();
#pragma unroll 1
  for (int t = 0; t < n_tiles; ++t) {
    if (t % kStage == 0) load_stage(t + kStage);
    const bf16_t* tb = lds + (t % (2 * kStage)) * kBuf;
    const int* pos = pos_lds_base + (t % (2 * kStage)) * BN;
    int mode = -1, live = 0, jt = 0, slots = 0;
    if (r0 < n) {
      if (t < n_win_tiles) {
        jt = jt0 + t * BN;
        if (!(jt > r_hi || jt + BN - 1 < r0 - window + 1))
          mode = ((jt + BN - 1 <= r0) && (jt >= r_hi - window + 1)) ? 0 : 1;
        live = (jt + 31 >= r0 - window + 1 ? 1 : 0) | (jt + 32 <= r_hi ? 2 : 0);      // of a tile that is not -1
      } else {
        // an entry counts once it has left the window of the wave's last row and needs no mask once it has left the first's
        slots = cnt - (t - n_win_tiles) * BN;
        int pv = pos[lane];
        pv = lane < slots ? pv : 0x7FFFFFFF;
        const uint64_t some = __builtin_amdgcn_ballot_w64(pv <= r_hi - window);
        live = ((uint32_t)some != 0u ? 1 : 0) | ((uint32_t)(some >> 32) != 0u ? 2 : 0);
        if (some != 0ull)
          mode = __builtin_amdgcn_ballot_w64(pv > r0 - window) == 0ull ? 0 : 2;
      }
    }
    mode = __builtin_amdgcn_readfirstlane(mode);
    live = __builtin_amdgcn_readfirstlane(live);
    // Two steps in sequence rather than if / else, so that the accumulators stay in place across the plain body.
    if (mode == 0) {
      compute_plain(tb);
      mode = -1;
    }
    asm volatile("" : "+s"(mode));
    if (mode == 1) compute(1, live, tb, pos, jt, slots);
    else if (mode == 2) compute(2, live, tb, pos, jt, slots);
    if (t % kStage == kStage - 1 || t == n_tiles - 1) {
      wait_loads();
      __syncthreads();               // the next stage is in LDS; everyone is done with this one
    }
  }

  // ---- epilogue: dQ = scale * acc, staged through LDS, rows stored coalesced ---------------------------------
  {
    bf16_t* orow = lds + (32 * wv + ql) * OS + 4 * hb;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        bf16x4 w4;
#pragma unroll
        for (int e = 0; e < 4; ++e) w4[e] = static_cast<bf16_t>(acc[db][4 * g4 + e] * A.scale);
        *reinterpret_cast<bf16x4*>(orow + 32 * db + 8 * g4) = w4;
      }
  }
  __syncthreads();
  {
    const int k_piece = tid % PPR, k_row = tid / PPR;
    bf16_t* obase = static_cast<bf16_t*>(A.dq) + ((int64_t)(lo + i0) * Hq + unit * HW) * D;
    const int64_t orow_stride = (int64_t)Hq * D;
#pragma unroll
    for (int p = 0; p < BM / RPP; ++p) {
      const int row = p * RPP + k_row, prow = HW == 1 ? row : row % 32, hd = HW == 1 ? 0 : row / 32;
      if (i0 + prow < n)
        *reinterpret_cast<u32x4*>(obase + prow * orow_stride + hd * D + k_piece * 8) =
            *reinterpret_cast<const u32x4*>(lds + row * OS + k_piece * 8);
    }
  }
}



// train_dkv_mfma_kernel<FAR>: one workgroup = 128 keys of one (sequence, KV head), 4 waves x 32 keys; a lane owns one
// key column.  It walks 64-query tiles of every query head of the group that can see its keys:
//   S[query, key]  = Q . K^T          A = Q tile rows from LDS, B = K fragment in registers
//   dP[query, key] = dO . V^T         A = dO tile rows from LDS, B = V fragment in registers
//   P = exp2(S c - lse[query]), dS = P (dP - delta[query])      lse, delta per row, read from LDS
//   dV^T[d, key] += dO^T . P          A = dO^T through the transposing LDS load, B = P from registers
//   dK^T[d, key] += Q^T . dS          A = Q^T through the transposing LDS load, B = dS from registers
// FAR = false ("band"): the keys are 128 consecutive positions, seen by the queries j .. j+window-1; the epilogue adds
// what the FAR pass left for keys that are candidates, rounds and stores dK, dV, and forms d logit and the counts.
// FAR = true: the keys are 128 consecutive entries of the compacted candidates (positions ascending), seen by the
// queries from position + window on; the fp32 sums go to a scratch array indexed like the compact segment.
template <int D, bool FAR>
__device__ __forceinline__ void dkv_body(const TrainArgs& A, int tiles_upper, float scale_log2e, float* far_dk,
                                         float* far_dv, int block, bf16_t* lds, float* stat_base) {
  LTEA_GEO(D);
  static_assert(2 * kStage * kBuf >= BM * OS, "epilogue staging must fit in the tile buffers");

  const int Hq = A.Hq, Hkv = A.Hkv, window = A.window, cap = A.budget;
  const int G = Hq / Hkv;
  int s, n, lo, h, j0 = 0, r_base = 0, cnt = 0;
  int chunk = 0;                          // FAR: which share of the query tiles this workgroup walks
  if (FAR) {
    // one workgroup per (128 compact entries, share of the query range): A.far_chunks shares of equal length keep
    // the workgroups short and alike; their partial sums go to one scratch slice each, which the band pass adds up
    // in a fixed order
    // The workgroups of one (head, share) read the same Q and dO tiles: order them so that they are neighbours, and
    // give each XCD a contiguous range of that order (workgroups are dealt round-robin to the 8 XCDs).
    const int per_head = (A.max_seqlen + BM - 1) / BM;
    const int n_far = A.n_seqs * Hkv * A.far_chunks * per_head;
    const int per_xcd = (n_far + 7) / 8;
    const int work = (block % 8) * per_xcd + block / 8;
    if (work >= n_far) return;            // padding workgroups of the combined launch
    const int rest = work / per_head;
    chunk = rest % A.far_chunks;
    const int hd = rest / A.far_chunks;
    r_base = (work - rest * per_head) * BM;
    s = hd / Hkv;
    h = hd - s * Hkv;
    cnt = A.ret_count[hd];
    if (r_base >= cnt) return;
    lo = A.cu[s];
    n = A.cu[s + 1] - lo;
  } else {
    // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of key tiles so that
    // neighbouring tiles of one head (which walk mostly the same Q and dO tiles) meet in the same L2.
    const int n_work = tiles_upper * Hkv;
    const int per_xcd = (n_work + 7) / 8;
    const int work = (block % 8) * per_xcd + block / 8;
    if (work >= n_work) return;
    h = work / tiles_upper;
    int tile;
    if (!locate_tile(A.cu, A.n_seqs, BM, work - h * tiles_upper, s, tile, lo, n)) return;
    j0 = tile * BM;
  }
  const int64_t head = (int64_t)s * Hkv + h;
  const int32_t* rp = A.ret_pos + head * cap;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ql = lane & 31, hb = lane >> 5;
  const bf16_t* q = static_cast<const bf16_t*>(A.q);
  const bf16_t* dout = static_cast<const bf16_t*>(A.dout);

  // ---- this lane's key: its K / V fragments and the range of queries [q_lo, q_hi) that saw it -----------------
  const int kloc = 32 * wv + ql;          // key index inside the workgroup
  int q_lo = 0, q_hi = 0, jpos = 0;
  const bf16_t *krow, *vrow;
  bool key_ok;
  if (FAR) {
    const int r = r_base + kloc;
    key_ok = r < cnt;
    const int rc = key_ok ? r : cnt - 1;
    jpos = rp[rc];
    krow = static_cast<const bf16_t*>(A.k_ret) + (head * cap + rc) * D;
    vrow = static_cast<const bf16_t*>(A.v_ret) + (head * cap + rc) * D;
    if (key_ok) { q_lo = jpos + window; q_hi = n; }
  } else {
    const int j = j0 + kloc;
    key_ok = j < n;
    jpos = key_ok ? j : n - 1;
    krow = static_cast<const bf16_t*>(A.k) + (int64_t)(lo + jpos) * A.kv_st + (int64_t)h * A.kv_sh;
    vrow = static_cast<const bf16_t*>(A.v) + (int64_t)(lo + jpos) * A.kv_st + (int64_t)h * A.kv_sh;
    if (key_ok) { q_lo = j; q_hi = j + window < n ? j + window : n; }
  }
  const unsigned q_span = (unsigned)(q_hi - q_lo);     // 0 for lanes without a key
  bf16x8 kreg[D / 16], vreg[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    kreg[ks] = *reinterpret_cast<const bf16x8*>(krow + 16 * ks + 8 * hb);
    vreg[ks] = *reinterpret_cast<const bf16x8*>(vrow + 16 * ks + 8 * hb);
  }

  // ---- query tiles the workgroup has to visit (the same for every query head of the group) --------------------
  int qt_first, qt_last;
  const int chunk_tiles = ((n + BN - 1) / BN + A.far_chunks - 1) / A.far_chunks;   // query tiles per share
  if (FAR) {
    qt_first = (rp[r_base] + window) / BN;            // positions ascend: the first entry is seen first
    qt_last = (n - 1) / BN;
    qt_first = qt_first > chunk * chunk_tiles ? qt_first : chunk * chunk_tiles;
    qt_last = qt_last < (chunk + 1) * chunk_tiles - 1 ? qt_last : (chunk + 1) * chunk_tiles - 1;
    if (qt_first > qt_last) return;                   // this share lies before the entries' first query: nothing to add
  } else {
    qt_first = j0 / BN;
    const int last_key = (j0 + BM < n ? j0 + BM : n) - 1;
    const int last_q = last_key + window - 1 < n - 1 ? last_key + window - 1 : n - 1;
    qt_last = last_q / BN;
  }
  const int n_qt = qt_last - qt_first + 1;
  const int n_iter = n_qt * G;

  const uint32_t q_row_bytes = (uint32_t)A.q_st * 2u, o_row_bytes = (uint32_t)(Hq * D) * 2u;
  const uint32_t q_bytes = (uint32_t)(n - 1) * q_row_bytes + (uint32_t)(D * 2);
  const uint32_t o_bytes = (uint32_t)(n - 1) * o_row_bytes + (uint32_t)(D * 2);
  const int ld_row = G_::RPI * wv + lane / PPR;        // global -> LDS as in the dQ role
  const uint32_t ld_col = (uint32_t)((lane % PPR) ^ both_ways_swizzle<D>(ld_row)) * 16u;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  const uint32_t stat_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)stat_base;
  auto load_tile = [&](int it) {
    const int g = it / n_qt, t = it - g * n_qt;
    const int hq = h * G + g;
    const int qt = (qt_first + t) * BN;
    const u32x4 rs_q = make_raw_rsrc(q + (int64_t)lo * A.q_st + (int64_t)hq * A.q_sh, q_bytes);
    const u32x4 rs_o = make_raw_rsrc(dout + ((int64_t)lo * Hq + hq) * D, o_bytes);
    const uint32_t dst = lds_base + (uint32_t)((it % (2 * kStage)) * kBuf * 2 + wv * 1024);
    uint32_t q_off = (uint32_t)(qt + ld_row) * q_row_bytes + ld_col, o_off = (uint32_t)(qt + ld_row) * o_row_bytes + ld_col;
#pragma unroll
    for (int i = 0; i < G_::IPW; ++i) {
      dma16(rs_q, dst + (uint32_t)(i * 4096), q_off);
      dma16(rs_o, dst + (uint32_t)(kTile * 2 + i * 4096), o_off);
      q_off += (uint32_t)(4 * G_::RPI) * q_row_bytes;
      o_off += (uint32_t)(4 * G_::RPI) * o_row_bytes;
    }
    if (wv < 2) {       // [-lse / scale of the 64 queries | their -delta], zeros past the sequence
      const float* src = A.delta + (int64_t)(wv == 0 ? Hq : 0) * A.total + (int64_t)hq * A.total + lo;
      dma4(make_raw_rsrc(src, (uint32_t)n * 4u), stat_lds + (uint32_t)(((it % (2 * kStage)) * 2 + wv) * BN * 4), (uint32_t)(qt + lane) * 4u);
    }
  };
  const Operands<D> op(lane);
  constexpr int NK = D / 16, ND = D / 32;

  f32x16 dva[ND], dka[ND];
#pragma unroll
  for (int db = 0; db < ND; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dva[db][r] = 0.f; dka[db][r] = 0.f; }

  // register r of a product is the tile's query 32*qb + 16*(r/8) + 8*hb + r%8; the products start from -lse / scale and -delta
  auto start_values = [&](const float* st, int qb) {
    f32x16 x;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const f32x4 y = *reinterpret_cast<const f32x4*>(st + 32 * qb + 16 * (r4 / 2) + 8 * hb + 4 * (r4 % 2));
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * r4 + e] = y[e];
    }
    return x;
  };

  auto compute_masked = [&](const bf16_t* tb, const float* st, int qt) {
#pragma unroll 1
    for (int qb = 0; qb < 2; ++qb) {
      // no key of the wave sees a query of the block
      if (__builtin_amdgcn_ballot_w64(q_span != 0u && q_lo < qt + 32 * qb + 32 && q_hi > qt + 32 * qb) == 0ull) continue;
      f32x16 sc = start_values(st, qb), dp = start_values(st + BN, qb);
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.rows(tb, qb, ks), kreg[ks], sc, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.rows(tb + kTile, qb, ks), vreg[ks], dp, 0, 0, 0);
      }
      bf16x8 pp[2], ps[2];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * qb + 16 * (r / 8) + 8 * hb + r % 8;
        float p = __builtin_amdgcn_exp2f(sc[r] * scale_log2e);
        p = ((unsigned)(qt + row - q_lo) < q_span) ? p : 0.f;
        pp[r / 8][r % 8] = static_cast<bf16_t>(p);
        ps[r / 8][r % 8] = static_cast<bf16_t>(p * dp[r]);
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int db = 0; db < ND; ++db) {
          dva[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.columns(tb + kTile, qb, kk, db), pp[kk], dva[db], 0, 0, 0);
          dka[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op.columns(tb, qb, kk, db), ps[kk], dka[db], 0, 0, 0);
        }
    }
  };

  // A tile that every key of the wave is seen by: 8 NK matrix instructions without a branch, arranged as in the dQ role.
  auto compute_plain = [&](const bf16_t* tb, const float* st) {
    auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
    auto operand = [&](int i) {          // of the tile's i-th matrix instruction
      const int blk = i / (2 * NK) % 2, j = i % (2 * NK);
      if (i < 4 * NK) return op.rows(tb + ((j & 1) ? kTile : 0), blk, j / 2);
      return op.columns(tb + ((j & 1) ? 0 : kTile), blk, j / (2 * ND), j / 2 % ND);
    };
    constexpr int kAhead = 8;            // operands on their way from LDS
    bf16x8 x[kAhead], p0[2], z0[2], p1[2], z1[2];
    f32x16 s0 = start_values(st, 0), d0 = start_values(st + BN, 0), s1, d1;
    float ep[16], ez[16];
    constexpr int per = 8 / NK;     // elements behind each of 2 NK matrix instructions
    auto exps = [&](int i, const f32x16& s, const f32x16& d) {
#pragma unroll
      for (int r = per * i; r < per * (i + 1); ++r) {
        ep[r] = __builtin_amdgcn_exp2f(s[r] * scale_log2e);
        ez[r] = ep[r] * d[r];
        asm volatile("" : "+v"(ep[r]), "+v"(ez[r]));      // here, not next to their first use
      }
    };
    auto pack = [&](int i, bf16x8 (&p)[2], bf16x8 (&z)[2]) {
#pragma unroll
      for (int r = per * i; r < per * (i + 1); ++r) {
        p[r / 8][r % 8] = static_cast<bf16_t>(ep[r]);
        z[r / 8][r % 8] = static_cast<bf16_t>(ez[r]);
      }
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) x[i] = operand(i);
    fence();
    static_for<8 * NK>([&](auto index) {
      constexpr int i = decltype(index)::value;
      bf16x8& a = x[i % kAhead];
      pin(a);
      constexpr int j = i % (2 * NK), ks = j / 2, db = j / 2 % ND, kk = j / (2 * ND);
      if constexpr (i < 2 * NK) {                            // products of block 0
        if (j & 1) d0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, vreg[ks], d0, 0, 0, 0);
        else s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kreg[ks], s0, 0, 0, 0);
      } else if constexpr (i < 4 * NK) {                     // products of block 1 / exponentials of block 0
        if (j & 1) d1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, vreg[ks], d1, 0, 0, 0);
        else s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kreg[ks], s1, 0, 0, 0);
      } else if constexpr (i < 6 * NK) {                     // dV, dK of block 0 / exponentials of block 1
        if (j & 1) dka[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, z0[kk], dka[db], 0, 0, 0);
        else dva[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p0[kk], dva[db], 0, 0, 0);
      } else {                                     // dV, dK of block 1
        if (j & 1) dka[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, z1[kk], dka[db], 0, 0, 0);
        else dva[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, p1[kk], dva[db], 0, 0, 0);
      }
      if constexpr (i + kAhead < 8 * NK) a = operand(i + kAhead);
      if (i == NK) { s1 = start_values(st, 1); d1 = start_values(st + BN, 1); }
      if constexpr (i >= 2 * NK && i < 4 * NK) {
        exps(j, s0, d0);
        if (j > 0) pack(j - 1, p0, z0);
        if (j == 2 * NK - 1) pack(j, p0, z0);
      } else if constexpr (i >= 4 * NK && i < 6 * NK) {
        exps(j, s1, d1);
        if (j > 0) pack(j - 1, p1, z1);
        if (j == 2 * NK - 1) pack(j, p1, z1);
      }
      fence();
    });
  };

  // a stage of tiles is computed while the next one is on its way into the other half of the buffers
  auto load_stage = [&](int it0) {
#pragma unroll
    for (int it = it0; it < it0 + kStage; ++it)
      if (it < n_iter) load_tile(it);
  };
  load_stage(0);
  wait_loads();
  __syncthreads();
#pragma unroll 1
  for (int it = 0; it < n_iter; ++it) {
    if (it % kStage == 0) load_stage(it + kStage);
    const bf16_t* tb = lds + (it % (2 * kStage)) * kBuf;
    const float* st = stat_base + (it % (2 * kStage)) * 2 * BN;
    const int qt = (qt_first + it % n_qt) * BN;
    // does any key of this wave see a query of the tile, and do all of them see all of it?
    const bool touches = q_span != 0u && q_lo < qt + BN && q_hi > qt;
    const bool covers = q_span != 0u && q_lo <= qt && q_hi >= qt + BN;
    int mode = __builtin_amdgcn_ballot_w64(touches) == 0ull ? -1 : (__builtin_amdgcn_ballot_w64(!covers) == 0ull ? 0 : 1);
    mode = __builtin_amdgcn_readfirstlane(mode);
    // Two steps in sequence rather than if / else, so that the accumulators stay in place across the plain body.
    if (mode == 0) {
      compute_plain(tb, st);
      mode = -1;
    }
    asm volatile("" : "+s"(mode));
    if (mode == 1) compute_masked(tb, st, qt);
    if (it % kStage == kStage - 1 || it == n_iter - 1) {
      wait_loads();
      __syncthreads();
    }
  }

  // ---- epilogue: accumulator register r of block db is feature d = 32*db + 8*(r/4) + 4*hb + r%4 of the lane's key ---
  if (FAR) {
    if (key_ok) {
      const int64_t slice = (int64_t)chunk * A.n_seqs * Hkv + head;
      float* fk = far_dk + (slice * cap + r_base + kloc) * D + 4 * hb;
      float* fv = far_dv + (slice * cap + r_base + kloc) * D + 4 * hb;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          f32x4 a, b;
#pragma unroll
          for (int e = 0; e < 4; ++e) { a[e] = dka[db][4 * g4 + e] * A.scale; b[e] = dva[db][4 * g4 + e]; }
          *reinterpret_cast<f32x4*>(fk + 32 * db + 8 * g4) = a;
          *reinterpret_cast<f32x4*>(fv + 32 * db + 8 * g4) = b;
        }
    }
    return;
  }
  // band: add the far part of candidate keys (their compact index by binary search over the ascending positions)
  int ridx = -1;
  if (key_ok && cap > 0) {
    int a = 0, b = A.ret_count[head];
    while (a < b) {
      const int mid = (a + b) >> 1;
      if (rp[mid] < jpos) a = mid + 1; else b = mid;
    }
    if (a < A.ret_count[head] && rp[a] == jpos) ridx = a;
  }
  // the shares of the query range in which the far pass wrote something for this entry's group of 128
  int c_first = 0, c_last = -1;
  if (ridx >= 0) {
    c_first = ((rp[ridx / BM * BM] + window) / BN) / chunk_tiles;
    c_last = ((n - 1) / BN) / chunk_tiles;
  }
  float ste = 0.f;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int d0 = 32 * db + 8 * g4 + 4 * hb;
      f32x4 fk = {0.f, 0.f, 0.f, 0.f}, fv = {0.f, 0.f, 0.f, 0.f};
      if (ridx >= 0) {
        for (int c = c_first; c <= c_last; ++c) {
          const int64_t slice = (int64_t)c * A.n_seqs * Hkv + head;
          const f32x4 a = *reinterpret_cast<const f32x4*>(far_dk + (slice * cap + ridx) * D + d0);
          const f32x4 b = *reinterpret_cast<const f32x4*>(far_dv + (slice * cap + ridx) * D + d0);
#pragma unroll
          for (int e = 0; e < 4; ++e) { fk[e] += a[e]; fv[e] += b[e]; }
        }
      }
      const bf16x4 v4 = *reinterpret_cast<const bf16x4*>(vrow + d0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dka[db][4 * g4 + e] = fmaf(dka[db][4 * g4 + e], A.scale, fk[e]);
        dva[db][4 * g4 + e] += fv[e];
        ste = fmaf(dva[db][4 * g4 + e], static_cast<float>(v4[e]), ste);
      }
    }
  ste = pair_sum(ste);
  {
    const float z = A.logits[(int64_t)h * A.total + lo + jpos];
    const bool above = key_ok && z > A.tau;
    if (key_ok && hb == 0) {
      const float r = 1.0f / (1.0f + expf(-z));
      A.dz[(int64_t)h * A.total + lo + jpos] = (ste + (above ? A.lambda[h] : 0.f)) * r * (1.0f - r);
    }
    const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(above && hb == 0));
    if (lane == 0 && c > 0) atomicAdd(&A.counts[s * Hkv + h], c);    // integer: order does not matter
  }
  bf16_t* outs[2] = {static_cast<bf16_t*>(A.dk), static_cast<bf16_t*>(A.dv)};
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
    bf16_t* orow = lds + kloc * OS + 4 * hb;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        bf16x4 w4;
#pragma unroll
        for (int e = 0; e < 4; ++e) w4[e] = static_cast<bf16_t>(which == 0 ? dka[db][4 * g4 + e] : dva[db][4 * g4 + e]);
        *reinterpret_cast<bf16x4*>(orow + 32 * db + 8 * g4) = w4;
      }
    __syncthreads();
    const int k_piece = tid % PPR, k_row = tid / PPR;
    bf16_t* obase = outs[which] + ((int64_t)(lo + j0) * Hkv + h) * D;
    const int64_t orow_stride = (int64_t)Hkv * D;
#pragma unroll
    for (int p = 0; p < BM / RPP; ++p) {
      const int row = p * RPP + k_row;
      if (j0 + row < n)
        *reinterpret_cast<u32x4*>(obase + row * orow_stride + k_piece * 8) =
            *reinterpret_cast<const u32x4*>(lds + row * OS + k_piece * 8);
    }
  }
}

// -delta = -<dO, O> and -lse / scale per (query, query head), from which the products of the other kernels start.  One
// workgroup = kDeltaTokens tokens of one head, heads fastest, PPR lanes per row: the results, [head][token], are written next
// to each other and all of a lane's rows are in flight together.
constexpr int kDeltaTokens = 128;
template <int D>
__global__ void __launch_bounds__(kThreads)
train_delta_mfma_kernel(TrainArgs A, float inv_scale) {
  constexpr int PPR = Geo<D>::PPR, RPP = Geo<D>::RPP, N = kDeltaTokens / RPP;
  const int hq = (int)(blockIdx.x % (unsigned)A.Hq);
  const int64_t tok0 = (int64_t)(blockIdx.x / (unsigned)A.Hq) * kDeltaTokens + threadIdx.x / PPR;
  const int piece = threadIdx.x % PPR;
  bf16x8 o8[N], d8[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int64_t tok = tok0 + i * RPP < A.total ? tok0 + i * RPP : A.total - 1;
    const int64_t at = (tok * A.Hq + hq) * D + piece * 8;
    o8[i] = *reinterpret_cast<const bf16x8*>(static_cast<const bf16_t*>(A.out) + at);
    d8[i] = *reinterpret_cast<const bf16x8*>(static_cast<const bf16_t*>(A.dout) + at);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fmaf(static_cast<float>(d8[i][e]), static_cast<float>(o8[i][e]), acc);
#pragma unroll
    for (int off = PPR / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
    const int64_t tok = tok0 + i * RPP;
    if (piece == 0 && tok < A.total) {
      const int64_t at = (int64_t)hq * A.total + tok;
      A.delta[at] = -acc;
      A.delta[(int64_t)A.Hq * A.total + at] = -A.lse[at] * inv_scale;
    }
  }
}

// One launch, two independent roles: the first far_blocks workgroups run the far pass of dK / dV (few, long-running:
// the candidates of early positions face almost every later query), the others compute dQ and fill the compute
// units that the far pass leaves idle.
// (D = 128 needs more than 256 registers per lane for the dK / dV role: one wave per SIMD there.)
template <int D, int HW>
__global__ void __launch_bounds__(kThreads, D == 64 ? 2 : 1)
train_dq_far_mfma_kernel(TrainArgs A, int tiles_upper, int n_work, float scale_log2e, float* far_dk, float* far_dv,
                         int far_blocks) {
  __shared__ __align__(1024) bf16_t lds[2 * kStage * Geo<D>::kBuf];  // for either role
  __shared__ __align__(256) float stat_lds[4 * kStage * BN];
  if ((int)blockIdx.x < far_blocks)
    dkv_body<D, true>(A, 0, scale_log2e, far_dk, far_dv, (int)blockIdx.x, lds, stat_lds);
  else
    dq_body<D, HW>(A, tiles_upper, n_work, scale_log2e, (int)blockIdx.x - far_blocks, lds, reinterpret_cast<int*>(stat_lds));
}

template <int D>
__global__ void __launch_bounds__(kThreads, D == 64 ? 2 : 1)
train_dkv_band_mfma_kernel(TrainArgs A, int tiles_upper, float scale_log2e, float* far_dk, float* far_dv) {
  __shared__ __align__(1024) bf16_t lds[2 * kStage * Geo<D>::kBuf];
  __shared__ __align__(256) float stat_lds[4 * kStage * BN];
  dkv_body<D, false>(A, tiles_upper, scale_log2e, far_dk, far_dv, (int)blockIdx.x, lds, stat_lds);
}

}  // namespace

// Rows are addressed with 32-bit byte offsets inside one sequence, and loaded in 16-byte pieces; lse / scale must not overflow.
bool train_mfma_supported(const TrainArgs& A, int D) {
  if (D != 64 && D != 128) return false;
  if (!(A.scale >= 1e-30f)) return false;
  if ((int64_t)A.max_seqlen * A.kv_st * 2 >= ((int64_t)1 << 31)) return false;
  if ((int64_t)A.max_seqlen * A.q_st * 2 >= ((int64_t)1 << 31)) return false;
  if ((int64_t)A.max_seqlen * A.Hq * D * 2 >= ((int64_t)1 << 31)) return false;
  if ((int64_t)A.budget * D * 2 >= ((int64_t)1 << 31)) return false;
  auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  return al16(A.dout) && al16(A.dq) && al16(A.dk) && al16(A.dv) && al16(A.out);
}

// delta, then [far pass of dK / dV | dQ] in one launch, then the band pass of dK / dV (which adds the far pass in).
// far_dk / far_dv: fp32 scratch, [far_chunks][n_seqs * Hkv][budget][D] each (only rows below ret_count are touched).
namespace {
template <int D, int HW>
hipError_t run_mfma(const TrainArgs& A, hipStream_t stream) {
  const float sl2 = A.scale * 1.4426950408889634f;
  const int64_t delta_blocks = (A.total + kDeltaTokens - 1) / kDeltaTokens * A.Hq;
  hipLaunchKernelGGL(train_delta_mfma_kernel<D>, dim3((unsigned)delta_blocks), dim3(kThreads), 0, stream, A, 1.0f / A.scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int per_head = (A.max_seqlen + BM - 1) / BM;
  int64_t far_blocks = A.budget > 0 ? (int64_t)A.n_seqs * A.Hkv * per_head * A.far_chunks : 0;
  far_blocks = (far_blocks + 7) / 8 * 8;      // keeps the dQ role's workgroup-to-XCD pattern
  const int64_t tiles_upper = (A.total + BM - 1) / BM + A.n_seqs;
  const int64_t dq_tiles = (A.total + BM / HW - 1) / (BM / HW) + A.n_seqs;
  const int64_t n_work = dq_tiles * (A.Hq / HW);
  const int64_t dq_blocks = (n_work + 7) / 8 * 8;
  hipLaunchKernelGGL((train_dq_far_mfma_kernel<D, HW>), dim3((unsigned)(far_blocks + dq_blocks)), dim3(kThreads), 0, stream, A,
                     (int)dq_tiles, (int)n_work, sl2, A.far_dk, A.far_dv, (int)far_blocks);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(train_dkv_band_mfma_kernel<D>, dim3((unsigned)((tiles_upper * A.Hkv + 7) / 8 * 8)), dim3(kThreads), 0, stream, A,
                     (int)tiles_upper, sl2, A.far_dk, A.far_dv);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_train_backward_mfma(const TrainArgs& A, int D, hipStream_t stream) {
  const bool by_head = (A.Hq / A.Hkv) % 4 == 0;      // one query head per wave (see dq_body)
  if (D == 64) return by_head ? run_mfma<64, 4>(A, stream) : run_mfma<64, 1>(A, stream);
  return by_head ? run_mfma<128, 4>(A, stream) : run_mfma<128, 1>(A, stream);
}

}  // namespace ltea
