// Scoring CNN of the LTE module (paper Section 3.1.1; Appendix A): fused single-layer bf16 path on MFMA.
//
//   z[h][j] = b_out[h] + sum_c w_out[h][c] * Swish( bias[h][c] + sum_{t,m} W[h][c][m][t] * x[j + (t-half)*dil][m] )
// with x = concat(key, value) of the token (2*D channels).  The contraction over (tap, channel) is a small
// GEMM per head: out^T[c, token] = W_t[c, :] . X^T[:, token + shift_t], run on v_mfma_f32_32x32x16_bf16 with
// the (zero-padded to 32) channels as MFMA rows and 32 tokens per wave as MFMA columns.  In the accumulator
// layout one lane owns one token, so bias, Swish and the output projection are per-lane work on the 16
// channel values it holds plus one exchange with the lane holding the other 16.
//
// Two launches:
//   score_weight_panels_kernel  re-lays the weights [Hkv][C][2D][k] once per call as tap-major panels
//                               [Hkv][k][32][2D] (channels zero-padded to 32) in the workspace, so that the main
//                               kernel can fetch a panel with coalesced 16-byte loads;
//   score_mfma_kernel           one workgroup = up to 8 consecutive tiles of one (sequence, KV head), 32 tokens per wave in
//                               a tile.  The weights of some input channels lie in LDS while all its tiles pass, one
//                               accumulator per tile: 128 channels (D = 64: all; D = 128: the keys', then the values'), or,
//                               for a workgroup of a single tile, 64.  A stage is 64 channels of a tile's rows with
//                               their halo of half*dil rows (zeros outside the sequence): it is multiplied out of one of
//                               two LDS buffers while the next one is stored into the other and the two after that are
//                               on their way to registers.  One barrier per stage; operand reads run three matrix
//                               instructions ahead of their use; a wave past the sequence's end multiplies nothing.
//
// What bounds it: the rows' way from memory, 64 channels (128 bytes) out of every token's 2 D Hkv: without the products of all
// but one tap it takes 194 of 231 us (119498 tokens in 16 sequences of 1024 to 16384, 16 heads of D = 128, k = 5) and 125 of 150
// (32768 tokens, 32 heads, k = 7), 5.0 and 4.3 TB/s where a linear read reaches 6.6.  Stages of a whole half of the channels (rows
// of 256 bytes) give 4 % of that, an order of heads that keeps an XCD's neighbouring nothing, non-temporal loads 2 % here and
// minus 15 % on 4 x 4096 tokens (32.2 -> 37.2 us: the attention's and the next call's rows then come from HBM).  What was slow
// before, with 128-token tiles of 128 channels in one buffer, the weights staged for groups of four tiles: at k = 7 one workgroup
// per CU, in lockstep through load, store and products (the matrix pipe busy for 57 of 197 us).  Before -> groups of up to 8 tiles,
// us per call: the two shapes above 259 -> 231 and 199 -> 150, 4 x 4096 x 16, k = 5 32.9 -> 31.9, D = 64, k = 7 30.0 -> 25.2.
// Short sequences: a workgroup's start and, at k >= 7, a CU's whole LDS for it made groups slower than that form (64 x 100 tokens,
// 32 heads: D = 64, k = 7 47.3 us then, 57.8 in groups; k = 1, for which there was a general instance only, 24.2 and 45.2); with single
// tiles, and idle waves leaving the matrix pipe to the others, 29.4 and 17.7.  One sequence of 100 tokens, 8 heads, k = 7: D = 64
// 8.0, 8.8, now 7.0, D = 128 11.4, 11.8, now 9.0.
// Tried: the weights beside every stage instead of resident (240 and 154 us); direct global-to-LDS rows of 32 channels,
// five stages deep, shared or private to the waves (274, 290 and 148, 150 us: pieces of 64 bytes).
#include <type_traits>

#include "ltea_common.h"
#include "ltea_kernels.h"
#include "score_dma.h"

namespace ltea {
namespace {

constexpr int CP = 32;        // channels padded to one MFMA tile
constexpr int SC = 64;        // input channels per stage: token rows of 128 bytes, all of them keys' or all values'
constexpr int kMaxRho = 4;    // largest half receptive field the token tile is sized for
constexpr int kMaxTaps = 2 * kMaxRho + 1;
constexpr int kMaxGroup = kScoreMfmaMaxGroup;      // tiles per workgroup
constexpr int weight_channels(int max_group) { return max_group == 1 ? 64 : 128; }     // whose weights are in LDS at a time
constexpr int stage_bytes(int waves) { return (32 * waves + 2 * kMaxRho) * SC * 2; }   // 32 tokens per wave and the halo
constexpr int tap_bytes(int channels) { return CP * channels * 2; }                    // one tap's weights

// panels[h][tap][c][m] = W[h][c][m][tap] for c < C, 0 for C <= c < 32
__global__ void __launch_bounds__(256)
score_weight_panels_kernel(const uint16_t* __restrict__ W, uint16_t* __restrict__ panels, int C, int C2, int ks,
                           int64_t total) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;   // over [Hkv][ks][32][C2]
  if (idx >= total) return;
  const int m = (int)(idx % C2);
  int64_t r = idx / C2;
  const int c = (int)(r % CP); r /= CP;
  const int tap = (int)(r % ks);
  const int64_t h = r / ks;
  panels[idx] = c < C ? W[((h * C + c) * C2 + m) * ks + tap] : (uint16_t)0;
}

// KS: the kernel size.  NW: waves; four where two workgroups share a CU's LDS (k <= 5, groups: 76 KB each; one hides the start of
// the other: 265 -> 231 us on the ragged shape above), eight where one fills it.  MG: most tiles per workgroup, kMaxGroup or 1
// (39 to 72 KB of LDS for k = 1 to 9: two to four workgroups per CU, by the registers too).
template <int D, int KS, int NW, int MG>
__global__ void __launch_bounds__(64 * NW, MG == 1 && KS < 5 ? 4 : 2)
score_mfma_kernel(const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int64_t st, int64_t sh,
                  const bf16_t* __restrict__ panels, const float* __restrict__ bias,
                  const bf16_t* __restrict__ w_out, const float* __restrict__ b_out, int C, int dil,
                  const int32_t* __restrict__ cu, int n_seqs, int Hkv, int64_t total, float* __restrict__ logits,
                  int group_tiles) {
  constexpr int kThreads = 64 * NW, TM = 32 * NW, kStageB = stage_bytes(NW);
  constexpr int HC = weight_channels(MG), kTapB = tap_bytes(HC);
  constexpr int C2 = 2 * D, NH = C2 / HC, SPT = HC / SC;      // input channels, passes over the tiles, stages per tile and pass
  extern __shared__ __align__(1024) unsigned char smem[];
  const int rho = (KS - 1) / 2 * dil;
  unsigned char* const w_lds = smem;                          // [tap][channel] rows of HC inputs
  unsigned char* const x_lds = smem + KS * kTapB;             // two stages of token rows
  float* const out_lds = reinterpret_cast<float*>(x_lds + 2 * kStageB);     // bias, output projection

  // heads fastest: workgroups that run together read neighbouring pieces of the same rows, and where the heads are a multiple
  // of the 8 XCDs an XCD sees the weights of its own heads only
  const int h = (int)(blockIdx.x % (unsigned)Hkv);
  const int tid = threadIdx.x, lane = tid & 63, ql = lane & 31, hb = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

  // weights of one pass: piece p of channel c's row to place p ^ (c & 15) or, in rows of half as many, p ^ ((c >> 1) & 7), so that the
  // operand reads of 16 consecutive channels at one piece cover all 64 banks
  constexpr int kWPieces = HC / 8, kWRows = kThreads / kWPieces;      // pieces per row, rows per pass of the threads
  auto w_place = [](int row) { return HC == 128 ? row & 15 : (row >> 1) & 7; };
  const int w_row = tid / kWPieces, w_piece = tid % kWPieces;
  const bf16_t* const w_src = panels + ((int64_t)h * KS * CP + w_row) * C2 + w_piece * 8;
  unsigned char* const w_dst = w_lds + w_row * (HC * 2) + ((w_piece ^ w_place(w_row)) << 4);
  u32x4 wreg[KS][CP / kWRows];
  auto load_weights = [&](int half) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KS; ++i)
#pragma unroll
      for (int j = 0; j < CP / kWRows; ++j)
        wreg[i][j] = *reinterpret_cast<const u32x4*>(w_src + ((int64_t)i * CP + j * kWRows) * C2 + half * HC);
  };
  auto store_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KS; ++i)
#pragma unroll
      for (int j = 0; j < CP / kWRows; ++j) *reinterpret_cast<u32x4*>(w_dst + i * kTapB + j * kWRows * (HC * 2)) = wreg[i][j];
  };
  load_weights(0);
  if (tid < CP) {
    const int c = tid < C ? tid : C - 1;         // unconditional loads, then select
    const float b_ld = bias[h * C + c], w_ld = to_f32(w_out[h * C + c]);
    out_lds[tid] = tid < C ? b_ld : 0.f;
    out_lds[CP + tid] = tid < C ? w_ld : 0.f;
  }
  const float bo = b_out[h];
  int grp, s, n, lo32;
  if (!locate_tile(cu, n_seqs, group_tiles * TM, (int)(blockIdx.x / (unsigned)Hkv), s, grp, lo32, n)) return;
  const int64_t lo = lo32;
  const int g0 = grp * group_tiles * TM;         // first token of this workgroup's tiles
  const int n_tiles = min((n - g0 + TM - 1) / TM, group_tiles);

  // Rows before the sequence start or past its end are outside the descriptors and arrive as zeros.  The descriptors start at
  // the first row this workgroup reads (the sequence start for the first group, whose halo rows then wrap to huge offsets)
  // and end at the last one or at the sequence end, so that 32-bit byte offsets only ever span one group of tiles.
  const uint32_t row_bytes = (uint32_t)st * 2u;
  const int base_row = g0 > 0 ? g0 - rho : 0;
  const int rows_here = min(n - base_row, n_tiles * TM + 2 * rho);
  const uint32_t seq_bytes = (uint32_t)(rows_here - 1) * row_bytes + (uint32_t)(D * 2);
  const int64_t base_el = (lo + base_row) * st + (int64_t)h * sh;
  const auto rs_k = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(k + base_el), 0, seq_bytes, 0x00020000);
  const auto rs_v = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(v + base_el), 0, seq_bytes, 0x00020000);
  // A thread brings one 16-byte piece of every kPassRows-th row.  Piece p of row r goes to place p ^ ((r >> 1) & 7), so that the operand
  // reads of 16 consecutive rows at one piece cover all 64 banks.
  constexpr int kPassRows = kThreads / 8, kPasses = TM / kPassRows;
  const int piece = tid & 7, r_in = tid >> 3;
  const uint32_t off0 = (uint32_t)(g0 - rho + r_in - base_row) * row_bytes + (uint32_t)piece * 16u;   // wraps for rows < 0
  const bool halo = r_in < 2 * rho;
  unsigned char* const x_dst = x_lds + r_in * (SC * 2) + ((piece ^ ((r_in >> 1) & 7)) << 4);
  u32x4 xreg[2][kPasses + 1];
  int ld_sub = 0, ld_tile = 0, ld_half = 0;      // the next stage to request
  auto request = [&](u32x4 (&x)[kPasses + 1]) __attribute__((always_inline)) {
    const int ch = ld_half * HC + ld_sub * SC;
    const bool is_v = ch >= D;
    const uint32_t off = off0 + (uint32_t)(ld_tile * TM) * row_bytes + (uint32_t)((is_v ? ch - D : ch) * 2);
#pragma unroll
    for (int i = 0; i <= kPasses; ++i) {
      const uint32_t at = i < kPasses || halo ? off + (uint32_t)(kPassRows * i) * row_bytes : 0xFFFFFFF0u;
      x[i] = is_v ? __builtin_amdgcn_raw_buffer_load_b128(rs_v, at, 0, 0) : __builtin_amdgcn_raw_buffer_load_b128(rs_k, at, 0, 0);
    }
    if (++ld_sub == SPT) {
      ld_sub = 0;
      if (++ld_tile == n_tiles) { ld_tile = 0; ++ld_half; }
    }
  };
  auto deposit = [&](const u32x4 (&x)[kPasses + 1], int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kPasses; ++i) *reinterpret_cast<u32x4*>(x_dst + buf * kStageB + i * (kPassRows * SC * 2)) = x[i];
    if (halo) *reinterpret_cast<u32x4*>(x_dst + buf * kStageB + kPasses * (kPassRows * SC * 2)) = x[kPasses];
  };
  const int n_stages = NH * n_tiles * SPT;

  f32x16 acc[MG];
#pragma unroll
  for (int t = 0; t < MG; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;

  // operands of one stage: steps of 16 channels of one tap, read kAhead steps before their products
  constexpr int NS = SC / 16, kAhead = 3, kOps = 4;
  static_assert(NS == kOps, "a step's operands have the place of its channels");
  const unsigned char* const a_base = w_lds + ql * (HC * 2);                  // channel ql
  const int a_swz = (w_place(ql) ^ hb) << 4;
  bf16x8 a_op[kOps], b_op[kOps];
  struct TapRow { const unsigned char* row; int swz; };
  auto multiply = [&](f32x16& sum, int buf, int sub) __attribute__((always_inline)) {
    auto tap_row = [&](int tap) __attribute__((always_inline)) {
      int row = 32 * wv + ql + tap * dil;
      asm volatile("" : "+v"(row));      // worked out here: kept for all taps these addresses are many registers
      return TapRow{x_lds + buf * kStageB + row * (SC * 2), (((row >> 1) & 7) ^ hb) << 4};
    };
    auto read_step = [&](const TapRow& at, int tap, int mc) __attribute__((always_inline)) {
      a_op[mc] = *reinterpret_cast<const bf16x8*>(a_base + tap * kTapB + (a_swz ^ (SC * 2 * sub + 32 * mc)));
      b_op[mc] = *reinterpret_cast<const bf16x8*>(at.row + (at.swz ^ (32 * mc)));
    };
    TapRow at = tap_row(0);
#pragma unroll
    for (int mc = 0; mc < kAhead; ++mc) read_step(at, 0, mc);
#pragma unroll
    for (int tap = 0; tap < KS; ++tap)
#pragma unroll
      for (int mc = 0; mc < NS; ++mc) {
        const int ahead = (mc + kAhead) % NS, tap_ahead = tap + (mc + kAhead) / NS;
        if (tap_ahead < KS) {
          if (ahead == 0) at = tap_row(tap_ahead);
          read_step(at, tap_ahead, ahead);
        }
        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a_op[mc], b_op[mc], sum, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
  };

  // Stage s: its rows are in buffer s & 1; those of s + 1 go to the other one, s + 2 and s + 3 are on their way.
  static_assert(SPT == 2 || MG == 1, "a stage's buffer and registers are those of its part of the tile, or of the only tile's pass");
  request(xreg[0]);
  request(xreg[1]);
  deposit(xreg[0], 0);
  if (n_stages > 2) request(xreg[0]);
  store_weights();
  __syncthreads();
  int at = 0;
  auto stage = [&](f32x16& sum, int t, auto buffer, int sub) __attribute__((always_inline)) {
    constexpr int S = decltype(buffer)::value;
    if (at + 1 < n_stages) deposit(xreg[S ^ 1], S ^ 1);
    if (at + 3 < n_stages) request(xreg[S ^ 1]);
    __builtin_amdgcn_sched_barrier(0);      // the requests leave before the products
    if (g0 + t * TM + 32 * wv < n) multiply(sum, S, sub);      // (a wave past the sequence's end has no tokens)
    __syncthreads();
    ++at;
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
#pragma unroll
  for (int half = 0; half < NH; ++half) {
    if (half > 0) {          // the other channels' weights; everyone is done with the ones before
      if (MG > 1) load_weights(half);
      store_weights();
      __syncthreads();
    }
    if constexpr (MG == 1) {
      if (half + 1 < NH) load_weights(half + 1);      // they arrive under this pass's products
      if (half % 2 == 0) stage(acc[0], 0, even, 0);
      else stage(acc[0], 0, odd, 0);
    } else {
#pragma unroll
      for (int t = 0; t < MG; ++t) {
        if (t < n_tiles) {     // uniform
          stage(acc[t], t, even, 0);
          stage(acc[t], t, odd, 1);
        }
      }
    }
  }

  // ---- epilogue: accumulator register r of lane half hb is channel 8*(r/4) + 4*hb + r%4 of token ql ----------
  float bs[16], wo[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    bs[r] = out_lds[8 * (r / 4) + 4 * hb + (r % 4)];
    wo[r] = out_lds[CP + 8 * (r / 4) + 4 * hb + (r % 4)];
  }
#pragma unroll
  for (int t = 0; t < MG; ++t) {
    if (t < n_tiles) {
      float z = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float y = acc[t][r] + bs[r];
        z = fmaf(y * __frcp_rn(1.0f + __expf(-y)), wo[r], z);
      }
      z += __shfl_xor(z, 32, kWave);
      const int j = g0 + t * TM + 32 * wv + ql;
      if (hb == 0 && j < n) logits[(int64_t)h * total + lo + j] = z + bo;
    }
  }
}

constexpr size_t lds_bytes(int ks, int waves, int group) {
  return (size_t)ks * tap_bytes(weight_channels(group)) + (size_t)2 * stage_bytes(waves) + 2 * CP * sizeof(float);
}

template <int D>
hipError_t run(const ltea_cfg& cfg, const ltea_cnn& cnn, const void* k, const void* v, int64_t st, int64_t sh,
               const SeqView& sv, float* logits, void* workspace, hipStream_t stream) {
  const int ks = cnn.kernel[0];
  const void* panels = cnn.panels;
  hipError_t e = hipSuccess;
  // the register-stationary kernel sorts unprepared weights itself (no launch for that) when they are 16-byte aligned
  if (panels == nullptr && score_reg_supported(cfg, cnn) && score_reg_takes_raw_weights(cnn))
    return launch_score_reg(cfg, cnn, k, v, st, sh, sv, logits, nullptr, stream);
  if (panels == nullptr) {            // not prepared by the caller: re-lay the weights into the workspace now
    e = launch_score_mfma_panels(cfg, cnn, workspace, stream);
    if (e != hipSuccess) return e;
    panels = workspace;
  }
  if (score_reg_supported(cfg, cnn)) return launch_score_reg(cfg, cnn, k, v, st, sh, sv, logits, panels, stream);
  const ScoreMfmaTiling tiling = score_mfma_tiling(score_batch(sv, cfg.Hkv), ks);
  auto launch = [&](auto taps, auto waves, auto tiles) {
    constexpr int KS = decltype(taps)::value, NW = decltype(waves)::value, MG = decltype(tiles)::value;
    constexpr size_t lds = lds_bytes(KS, NW, MG);
    const int64_t span = (int64_t)tiling.tiles * 32 * NW, groups_upper = (sv.total_tokens + span - 1) / span + sv.n_seqs;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&score_mfma_kernel<D, KS, NW, MG>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return;
    hipLaunchKernelGGL((score_mfma_kernel<D, KS, NW, MG>), dim3((unsigned)(groups_upper * cfg.Hkv)), dim3(64 * NW), lds, stream,
                       static_cast<const bf16_t*>(k), static_cast<const bf16_t*>(v), st, sh,
                       static_cast<const bf16_t*>(panels), cnn.bias[0], static_cast<const bf16_t*>(cnn.w_out),
                       cnn.b_out, cnn.c_out[0], cnn.dilation[0], sv.cu_seqlens, sv.n_seqs, cfg.Hkv, sv.total_tokens, logits,
                       tiling.tiles);
    e = hipGetLastError();
  };
  auto launch_taps = [&](auto taps) {
    constexpr int KS = decltype(taps)::value;
    if constexpr (KS > 3) {
      if (!tiling.single) {
        constexpr int kWaves = KS <= 5 ? 4 : 8;      // score_mfma_tiling's
        return launch(taps, std::integral_constant<int, kWaves>{}, std::integral_constant<int, kMaxGroup>{});
      }
    }
    launch(taps, std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
  };
  if (ks == 1) launch_taps(std::integral_constant<int, 1>{});
  else if (ks == 7) launch_taps(std::integral_constant<int, 7>{});
  else if (ks == 9) launch_taps(std::integral_constant<int, 9>{});
  else if constexpr (D == 128) {      // D = 64: the register-stationary kernel takes k = 3 and 5
    if (ks == 3) launch_taps(std::integral_constant<int, 3>{});
    else launch_taps(std::integral_constant<int, 5>{});
  }
  return e;
}

}  // namespace

bool score_mfma_supported(const ltea_cfg& cfg, const ltea_cnn& cnn) {
  if (cfg.dtype != LTEA_BF16 || cnn.n_layers != 1 || cnn.c_out[0] > CP) return false;
  if (cfg.D != 64 && cfg.D != 128) return false;
  if ((cnn.kernel[0] - 1) / 2 * cnn.dilation[0] > kMaxRho) return false;
  static_assert(kMaxGroup * 256 + 2 * kMaxRho + 16 <= kScoreRowsPerDescriptor, "rows one workgroup addresses");
  return cnn.kernel[0] <= kMaxTaps;
}

hipError_t launch_score_mfma_panels(const ltea_cfg& cfg, const ltea_cnn& cnn, void* panels, hipStream_t stream) {
  if (score_reg_supported(cfg, cnn)) return launch_score_reg_panels(cfg, cnn, panels, stream);   // its own order, same size
  const int ks = cnn.kernel[0], C2 = 2 * cfg.D;
  const int64_t panel_elems = (int64_t)cfg.Hkv * ks * CP * C2;
  hipLaunchKernelGGL(score_weight_panels_kernel, dim3((unsigned)((panel_elems + 255) / 256)), dim3(256), 0, stream,
                     static_cast<const uint16_t*>(cnn.w[0]), static_cast<uint16_t*>(panels), cnn.c_out[0], C2, ks,
                     panel_elems);
  return hipGetLastError();
}

size_t score_mfma_workspace(const ltea_cfg& cfg, const ltea_cnn& cnn) {
  return (size_t)cfg.Hkv * cnn.kernel[0] * CP * 2 * cfg.D * sizeof(uint16_t);
}

hipError_t launch_score_mfma(const ltea_cfg& cfg, const ltea_cnn& cnn, const void* k, const void* v, int64_t st,
                             int64_t sh, const SeqView& sv, float* logits, void* workspace, hipStream_t stream) {
  if (sv.total_tokens == 0) return hipSuccess;
  return cfg.D == 64 ? run<64>(cfg, cnn, k, v, st, sh, sv, logits, workspace, stream)
                     : run<128>(cfg, cnn, k, v, st, sh, sv, logits, workspace, stream);
}

}  // namespace ltea
