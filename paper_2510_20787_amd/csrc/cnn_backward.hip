// Backward of the scoring CNN of the LTE module (paper Section 3.1.1; trained through the gradient of the logits
// that Section 3.1.2 defines): from d(loss)/d(logit) to the gradients of every conv weight, bias, the output
// projection and the input features.  fp32-accurate arithmetic for any depth and either storage type, as LDS-tiled
// products on the fp32 matrix instruction, or, on bf16 storage where one operand is a bf16 value, on the bf16 one with
// the fp32 operand split into three bf16 terms.  The module is small next to the attention (paper stack: 65 kflop
// per token-head forward).  Everything is summed in a fixed order: same bits every run.
//
//   1. forward again, keeping the pre-activations y_l and the activations a_l = silu(y_l) of every layer
//      (fp32 [Hkv][T][C_l] each); the features of layer 0 are copied to a dense fp32 array first unless the bf16
//      kernels read k / v themselves;
//   2. d y_L = dz * w_out * silu'(y_L);  d w_out = sum_t dz * silu(y_L),  d b_out = sum_t dz   (the last layer's forward
//      launch: neither its pre-activations nor its activations go to memory);
//   3. for l = L .. 1:  d bias_l = sum_t d y_l;
//                       d W_l[c][m][tap] = sum_t d y_l[t][c] * a_{l-1}[t + off(tap)][m]      (inside the sequence)
//                       d a_{l-1}[t][m]  = sum_{tap, c} W_l[c][m][tap] * d y_l[t - off(tap)][c]
//                       d y_{l-1} = d a_{l-1} * silu'(y_{l-1})        (l > 1)   or   dk, dv = d a_0   (l = 1).
// Sums over tokens are taken in two stages: per chunk (weights) or TMC tokens (the column sums, by the
// workgroup that computes the column) into a partial array, then over the chunks.
#include <type_traits>

#include "ltea_common.h"
#include "ltea_kernels.h"
#include "rope_dev.h"
#include "mfma_tiles.h"

namespace ltea {
namespace {

constexpr int kTokChunk = 512;   // most tokens per partial of the weight products

__device__ __forceinline__ float silu_grad_f32(float y) {
  const float s = 1.0f / (1.0f + expf(-y));
  return s * (1.0f + y * (1.0f - s));
}

// Layer-0 input as a dense fp32 array: a0[h][t][m] = concat(key, value) features of token t, moved in 16-byte pieces of
// the storage type (rows of D elements are whole pieces).
template <typename T>
__global__ void __launch_bounds__(256)
features_kernel(const T* __restrict__ k, const T* __restrict__ v, int64_t stride_tok, int64_t stride_head, int D,
                int64_t total, float* __restrict__ a0) {
  constexpr int EPP = Elems<T>::N;
  const int h = blockIdx.y;
  const int pieces = 2 * D / EPP;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t tok = idx / pieces;
  const int m = (int)(idx - tok * pieces) * EPP;
  if (tok >= total) return;
  const T* src = (m < D ? k : v) + tok * stride_tok + (int64_t)h * stride_head + (m < D ? m : m - D);
  float x[EPP];
  Elems<T>::unpack(*reinterpret_cast<const u32x4*>(src), x);
  float4* dst = reinterpret_cast<float4*>(a0 + ((int64_t)h * total + tok) * 2 * D + m);
#pragma unroll
  for (int i = 0; i < EPP / 4; ++i) dst[i] = make_float4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
}

// What the launches after it read besides the inputs, in one launch.  blockIdx.y < n_layers: the weights of that layer in
// the orders its kernels contract over, those that are not null: fp32 wf[h][tap][m][c] (over the input channels m: the
// forward) and wb[h][tap][c][m] (over the output channels c: towards the input), and the same two orders, wqf and wq, in the
// storage type (operands of the bf16 matrix instruction).  blockIdx.y == n_layers: seq_lo[t], seq_hi[t], the bounds of the
// sequence token t belongs to.
struct LayerPanels { const void* w; float *wf, *wb; void *wq, *wqf; int cin, cout, ks; int64_t n; };
struct PrepareArgs {
  LayerPanels layer[LTEA_MAX_CNN_LAYERS];
  int n_layers;
  const int32_t* cu;
  int n_seqs;
  int64_t total;
  int32_t *seq_lo, *seq_hi;
};
template <typename T>
__global__ void __launch_bounds__(256)
prepare_kernel(const PrepareArgs A) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if ((int)blockIdx.y == A.n_layers) {
    if (i >= A.total) return;
    const int s = find_sequence(A.cu, A.n_seqs, i);
    A.seq_lo[i] = A.cu[s];
    A.seq_hi[i] = A.cu[s + 1];
    return;
  }
  const LayerPanels& L = A.layer[blockIdx.y];
  if (i >= L.n) return;                                          // over [h][c][m][tap]
  const int tap = (int)(i % L.ks);
  const int m = (int)((i / L.ks) % L.cin);
  const int c = (int)((i / ((int64_t)L.ks * L.cin)) % L.cout);
  const int64_t h = i / ((int64_t)L.ks * L.cin * L.cout);
  const T w = static_cast<const T*>(L.w)[i];
  const int64_t fwd = ((h * L.ks + tap) * L.cin + m) * L.cout + c, back = ((h * L.ks + tap) * L.cout + c) * L.cin + m;
  if (L.wf != nullptr) L.wf[fwd] = to_f32(w);
  if (L.wb != nullptr) L.wb[back] = to_f32(w);
  if (L.wq != nullptr) static_cast<T*>(L.wq)[back] = w;
  if (L.wqf != nullptr) static_cast<T*>(L.wqf)[fwd] = w;
}

// The fp32 products below run on v_mfma_f32_32x32x2_f32 (fp32 operands, two contraction steps per instruction: lane l
// supplies row / column l % 32 of step l / 32), their operands staged through LDS.  Weight products: up to TM input
// channels x TN output channels per workgroup in 32 x 32 pieces per wave; conv products: TN outputs wide.
constexpr int TM = 64, TN = 64;
// conv products: TMC tokens per workgroup (two 32-token sub-tiles per wave), contraction slices of KCC channels, up
// to GT taps per stage whose rows reach at most HALO past the tile; LDS row strides RSA / RSB keep the 16-byte operand
// reads of 16 neighbouring lanes, and the two lane halves' weight reads, on different banks
constexpr int TMC = 128, KCC = 16, HALO = 64, GT = 3, RSA = KCC + 4, RSB = 72;
constexpr int A_ROWS = TMC + HALO, PA = A_ROWS * (KCC / 4) / 256, PB = GT * KCC * (TN / 4) / 256;
static_assert(A_ROWS * (KCC / 4) % 256 == 0 && GT * KCC * (TN / 4) % 256 == 0, "whole quads per thread");
constexpr int KCW = 32, PERW = KCW * TM / 256;   // weight products: tokens per contraction slice

// row[x .. x+3] of a readable row of `limit` floats, loaded unconditionally from addresses clamped into the row, with
// a 4-bit mask of the elements that count (those below the limit, none when !ok).  The caller zeroes the others where
// it consumes the quad, so that a thread's loads of a stage are all in flight together and none is waited for before
// then.  VEC: limit % 4 == 0 and the row starts on a 16-byte boundary, so a quad is inside or outside as a whole.
template <bool VEC>
__device__ __forceinline__ float4 load_quad(const float* __restrict__ row, int x, int limit, bool ok, unsigned& mask4) {
  if constexpr (VEC) {
    mask4 = (ok && x < limit) ? 0xFu : 0u;
    return *reinterpret_cast<const float4*>(row + min(x, limit - 4));
  } else {
    const int last = limit - 1;
    mask4 = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) mask4 |= (ok && x + c < limit) ? 1u << c : 0u;
    return make_float4(row[min(x, last)], row[min(x + 1, last)], row[min(x + 2, last)], row[min(x + 3, last)]);
  }
}

// v if keep, else zero.  The empty asm makes the loaded value needed either way, so the load stays where it was issued
// instead of moving under a condition (and being waited for at once).
__device__ __forceinline__ float masked_value(float v, bool keep) {
  asm volatile("" : "+v"(v));
  return keep ? v : 0.f;
}

// The quad with the elements outside the mask zeroed.  The empty asm makes the loaded value needed whatever the mask
// says, so the load stays where it was issued instead of moving under a condition.
__device__ __forceinline__ float4 masked_quad(float4 v, unsigned mask4) {
  asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
  return make_float4(mask4 & 1u ? v.x : 0.f, mask4 & 2u ? v.y : 0.f, mask4 & 4u ? v.z : 0.f, mask4 & 8u ? v.w : 0.f);
}

// Sums over a workgroup's TMC tokens of NS values per output column, from the sums of a lane's own rows, in a fixed order:
// the two lane halves, then the waves that share the columns (four; two when a row of waves is 64 columns wide).  The
// result is in the threads tid < 64 (NARROW: 32), column tid.  All threads of the workgroup call it; red: LDS that is free.
template <int NS, bool NARROW>
__device__ __forceinline__ void tile_column_sums(float (&x)[NS], float* red, int wv, int lane) {
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    x[i] = pair_sum(x[i]);
    if (lane < 32) red[i * 128 + wv * 32 + lane] = x[i];
  }
  __syncthreads();
  if (wv == 0) {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const float* r = red + i * 128 + lane;
      x[i] = NARROW ? ((r[0] + r[32 * (lane < 32)]) + r[64 * (lane < 32)]) + r[96 * (lane < 32)] : r[0] + r[64];
    }
  }
}

// Of the last layer's forward launch: the output projection and its backward.  dz [Hkv][T], w_out [Hkv][C]; part_* get the
// sums over the workgroup's tokens ([tile of TMC tokens][Hkv][C], part_bout [tile][Hkv]).
template <typename T> struct OutProj {
  const float* dz;            // null: not the last layer
  const T* w_out;
  float *part_b, *part_wout, *part_bout;
};

// A workgroup's tokens of an array [Hkv][T][N], as a lane of the epilogues below sees them: accumulator register r of
// sub-tile u is row 32 u + 8 (r / 4) + r % 4 below the lane's own (row0), column n.  A row past the array's end or a column
// past N is outside the descriptor: its load gives zero and its store goes nowhere, so that a lane's elements are one straight
// run of independent chains (exponentials, divisions) without a branch or a 64-bit product in each.  (With both, the first
// layer's forward was 2025 vector instructions per wave, of which 1440 were the 32 elements.)
template <int U> struct TileColumn {
  static constexpr uint32_t kOutside = 0x80000000u;      // at or past the largest descriptor: 128 rows of 64 * 65536 columns
  int h, rows, row0, n, N;
  bool n_ok;
  int64_t first;                                         // h * T + the tile's first token

  __device__ __forceinline__ TileColumn(int h_, int64_t total, int64_t t0, int row0_, int n_, int N_)
      : h(h_), rows((int)(total - t0 < TMC ? total - t0 : TMC)), row0(row0_), n(n_), N(N_), n_ok(n_ < N_), first(h_ * total + t0) {}
  static __device__ __forceinline__ constexpr int row_of(int u, int r) { return 32 * u + 8 * (r / 4) + r % 4; }
  __device__ __forceinline__ bool inside(int u, int r) const { return row0 + row_of(u, r) < rows; }
  __device__ __forceinline__ uint32_t bytes() const { return (uint32_t)rows * (uint32_t)N * 4u; }
  __device__ __forceinline__ uint32_t base() const { return n_ok ? ((uint32_t)row0 * (uint32_t)N + (uint32_t)n) * 4u : kOutside; }
  __device__ __forceinline__ uint32_t at(uint32_t base, int u, int r) const { return base + (uint32_t)row_of(u, r) * (uint32_t)N * 4u; }
  template <class P> __device__ __forceinline__ auto rows_of(P* p) const {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p) + first * N, 0, bytes(), 0x00020000);
  }
};

// From the pre-activations y of a lane's tokens of its column to d y and the column's sums.
template <int U, bool NARROW, typename T>
__device__ __forceinline__ void out_proj_backward(const OutProj<T>& P, const f32x16 (&acc)[U], float bv, const TileColumn<U>& C,
                                                  int Hkv, float* dpre, float* red, int wv, int lane) {
  const float wo = C.n_ok ? to_f32(P.w_out[(int64_t)C.h * C.N + C.n]) : 0.f;
  const float* const dz = P.dz + C.first;
  const auto rs_d = C.rows_of(dpre);
  const uint32_t base = C.base();
  float sum[3] = {0.f, 0.f, 0.f};        // of d y, dz * silu(y), dz
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float g[16];                         // all requested before the first is used
#pragma unroll
    for (int r = 0; r < 16; ++r) g[r] = dz[(uint32_t)min(C.row0 + C.row_of(u, r), C.rows - 1)];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float y = acc[u][r] + bv;
      const float den = 1.0f + expf(-y), s = 1.0f / den;
      const float d = g[r] * wo * (s * (1.0f + y * (1.0f - s)));
      const bool keep = C.inside(u, r);
      sum[0] += keep ? d : 0.f;
      sum[1] += keep ? g[r] * (y / den) : 0.f;
      sum[2] += keep ? g[r] : 0.f;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d), rs_d, C.at(base, u, r), 0, 0);
      if (r % 4 == 3) {                  // four chains side by side, and their sums taken: 32 would not fit the registers
        asm volatile("" : "+v"(sum[0]), "+v"(sum[1]), "+v"(sum[2]));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  tile_column_sums<3, NARROW>(sum, red, wv, lane);
  const int col = (int)blockIdx.y * 64 + lane;
  if (wv == 0 && lane < (NARROW ? 32 : 64) && col < C.N) {
    const int64_t row = (int64_t)blockIdx.x * Hkv + C.h;
    P.part_b[row * C.N + col] = sum[0];
    P.part_wout[row * C.N + col] = sum[1];
    if (col == 0) P.part_bout[row] = sum[2];
  }
}

// What a forward launch does with its products: pre-activations and activations, or the output projection's backward.
template <int U, bool NARROW, typename T>
__device__ __forceinline__ void forward_result(const OutProj<T>& P, const f32x16 (&acc)[U], const float* bias,
                                               const TileColumn<U>& C, int Hkv, float* out0, float* out1, float* red, int wv,
                                               int lane) {
  const float bv = C.n_ok ? bias[(int64_t)C.h * C.N + C.n] : 0.f;
  if (P.dz != nullptr) {
    out_proj_backward<U, NARROW>(P, acc, bv, C, Hkv, out0, red, wv, lane);
    return;
  }
  const auto rs0 = C.rows_of(out0), rs1 = C.rows_of(out1);
  const uint32_t base = C.base();
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float y = acc[u][r] + bv;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(y), rs0, C.at(base, u, r), 0, 0);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(silu_f32(y)), rs1, C.at(base, u, r), 0, 0);
      if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);      // four chains side by side, not 32: registers
    }
}

// d y of the layer below from d a (acc), and its column sums over the workgroup's tokens.
template <int U, bool NARROW>
__device__ __forceinline__ void hidden_backward(const f32x16 (&acc)[U], const TileColumn<U>& C, int Hkv, const float* pre_prev,
                                                float* dpre, float* part_b, float* red, int wv, int lane) {
  const auto rs_p = C.rows_of(pre_prev), rs_d = C.rows_of(dpre);
  const uint32_t base = C.base();
  float sum[1] = {0.f};
  // per sub-tile, all of the lane's pre-activations are requested before the first is used
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float pp[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) pp[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_p, C.at(base, u, r), 0, 0));
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float d = acc[u][r] * silu_grad_f32(pp[r]);
      sum[0] += C.inside(u, r) ? d : 0.f;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(d), rs_d, C.at(base, u, r), 0, 0);
      if (r % 4 == 3) {
        asm volatile("" : "+v"(sum[0]));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  tile_column_sums<1, NARROW>(sum, red, wv, lane);
  const int col = (int)blockIdx.y * 64 + lane;
  if (wv == 0 && lane < (NARROW ? 32 : 64) && col < C.N) part_b[((int64_t)blockIdx.x * Hkv + C.h) * C.N + col] = sum[0];
}

// out[t][n] = sum_tap sum_k in[t + sign * off(tap)][k] * wt[tap][k][n]   (rows outside t's sequence count as zero)
// for one head, as a tiled fp32 product: TMC tokens x TN outputs per workgroup.  A stage brings one contraction slice
// of KCC channels into LDS: the input rows of the tile plus the extra rows that a group of up to GT taps reaches
// (at most HALO), and those taps' weight rows; every staged input row then serves all taps of the group.  Whether a
// tap's row lies in the token's own sequence is decided where the operand is read.  What is done with the result:
//   mode 0 (forward)          pre = out + bias, act = silu(pre); the last layer: d pre (out0) and the output projection's sums
//   mode 1 (hidden backward)  dpre_out = out * silu'(pre_prev), and its column sums over the tile's tokens (part_b)
//   mode 2 (input backward)   dk / dv [T][Hkv][D] of the storage type (n < D: key part)
template <typename T, bool VEC, bool NARROW>
__global__ void __launch_bounds__(256, 4)
conv_product_kernel(const float* __restrict__ in, const float* __restrict__ wt, int K, int N, int ks, int dil, int sign,
                    const int32_t* __restrict__ seq_lo, const int32_t* __restrict__ seq_hi, int64_t total, int Hkv,
                    int mode, const float* __restrict__ bias, const float* __restrict__ pre_prev,
                    float* __restrict__ out0, float* __restrict__ out1, T* __restrict__ dk, T* __restrict__ dv, int D,
                    const OutProj<T> proj, float* __restrict__ part_b) {
  __shared__ __align__(16) float a_s[A_ROWS][RSA];     // [staged input row][channel of the slice]
  __shared__ __align__(16) float b_s[GT * KCC][RSB];   // [tap of the group][channel of the slice][output]
  const int h = blockIdx.z;
  const int64_t t0 = (int64_t)blockIdx.x * TMC;
  const int n0 = blockIdx.y * TN;
  const int tid = threadIdx.x;
  const float* in_h = in + (int64_t)h * total * K;
  const float* wt_h = wt + (int64_t)h * ks * K * N;
  const int half = (ks - 1) / 2;
  const int lane = tid & 63, wv = tid >> 6, ql = lane & 31, hb = lane >> 5;
  // Wave roles.  Wide: the waves form 2 x 2, each with two 32-token sub-tiles and one 32-column half of the outputs.
  // NARROW (N <= 32): the four waves take 32 tokens each and the one column half there is.
  constexpr int U = NARROW ? 1 : 2;
  const int row0 = NARROW ? 32 * wv : 64 * (wv >> 1), col0 = NARROW ? 0 : 32 * (wv & 1);
  // the wave's two token rows per lane, and the bounds of their sequences
  int64_t tok[U];
  int lo[U], hi[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    tok[u] = t0 + row0 + 32 * u + ql;
    const bool ok = tok[u] < total;
    lo[u] = ok ? seq_lo[tok[u]] : 0;
    hi[u] = ok ? seq_hi[tok[u]] : 0;
  }
  f32x16 acc[U];         // wide: two token sub-tiles of 32 per wave, every weight operand read serves two MFMAs
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[u][r] = 0.f;
  const int per_group = min(GT, 1 + HALO / dil);       // taps whose rows fit the staged halo
  const int groups = (ks + per_group - 1) / per_group;
  const int slices = (K + KCC - 1) / KCC, stages = groups * slices;
  // of a stage: first tap, number of taps, and the offset of the first staged row from the tile's first token
  auto stage_taps = [&](int stage, int& tap0, int& ntap, int& k0, int& base_off) {
    const int g = stage / slices;
    k0 = (stage - g * slices) * KCC;
    tap0 = g * per_group;
    ntap = min(per_group, ks - tap0);
    base_off = sign > 0 ? (tap0 - half) * dil : -(tap0 + ntap - 1 - half) * dil;
  };
  // The next stage's operands are fetched into registers while the current one is multiplied.
  float4 ra[PA], rb[PB];
  unsigned mask_a, mask_b;       // four bits per quad: which of its elements count
  auto fetch = [&](int stage) {
    int tap0, ntap, k0, base_off;
    stage_taps(stage, tap0, ntap, k0, base_off);
    const int rows = TMC + (ntap - 1) * dil;
    mask_a = mask_b = 0u;
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      const int e = tid + 256 * i, row = e / (KCC / 4), q = e % (KCC / 4);
      const int64_t p = t0 + row + base_off;
      const bool ok = row < rows && p >= 0 && p < total;
      unsigned m4;
      ra[i] = load_quad<VEC>(in_h + (ok ? p : 0) * K, k0 + 4 * q, K, ok, m4);
      mask_a |= m4 << (4 * i);
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      const int e = tid + 256 * i, jrow = e / (TN / 4), q = e % (TN / 4);
      const int j = jrow / KCC, kk = jrow % KCC;
      const bool ok = j < ntap && k0 + kk < K;
      unsigned m4;
      rb[i] = load_quad<VEC>(wt_h + (ok ? ((int64_t)(tap0 + j) * K + k0 + kk) * N : 0), n0 + 4 * q, N, ok, m4);
      mask_b |= m4 << (4 * i);
    }
  };
  fetch(0);
  for (int stage = 0; stage < stages; ++stage) {
    __syncthreads();     // the previous stage's tiles are no longer read
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      const int e = tid + 256 * i;
      *reinterpret_cast<float4*>(&a_s[e / (KCC / 4)][4 * (e % (KCC / 4))]) = masked_quad(ra[i], mask_a >> (4 * i));
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      const int e = tid + 256 * i;
      *reinterpret_cast<float4*>(&b_s[e / (TN / 4)][4 * (e % (TN / 4))]) = masked_quad(rb[i], mask_b >> (4 * i));
    }
    __syncthreads();
    int tap0, ntap, k0, base_off;
    stage_taps(stage, tap0, ntap, k0, base_off);
    if (stage + 1 < stages) fetch(stage + 1);
    const int kgroups = (min(KCC, K - k0) + 7) / 8;
    for (int j = 0; j < ntap; ++j) {
      const int off = sign * (tap0 + j - half) * dil;
      const int shift = off - base_off;                 // 0 .. (ntap-1)*dil
      bool valid[U];
#pragma unroll
      for (int u = 0; u < U; ++u) valid[u] = tok[u] + off >= lo[u] && tok[u] + off < hi[u];
      // Lane half hb takes channels 8g + 4hb .. 8g + 4hb + 3 of each group of eight, one per MFMA, from both operands.
      for (int g = 0; g < kgroups; ++g) {
        float4 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          a[u] = *reinterpret_cast<const float4*>(&a_s[row0 + 32 * u + ql + shift][8 * g + 4 * hb]);
        const float* bp = &b_s[j * KCC + 8 * g + 4 * hb][col0 + ql];
        const float b0 = bp[0], b1 = bp[RSB], b2 = bp[2 * RSB], b3 = bp[3 * RSB];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = masked_quad(a[u], valid[u] ? 0xFu : 0u);
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u].x, b0, acc[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u].y, b1, acc[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u].z, b2, acc[u], 0, 0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u].w, b3, acc[u], 0, 0, 0);
      }
    }
  }
  // accumulator register r of lane half hb: token row 8*(r/4) + 4*hb + r%4 of the sub-tile, output column ql
  const int n = n0 + col0 + ql;
  const TileColumn<U> column(h, total, t0, row0 + 4 * hb, n, N);
  if (mode == 0) {
    forward_result<U, NARROW>(proj, acc, bias, column, Hkv, out0, out1, &a_s[0][0], wv, lane);
  } else if (mode == 1) {
    hidden_backward<U, NARROW>(acc, column, Hkv, pre_prev, out0, part_b, &a_s[0][0], wv, lane);
  } else {
    T* dst = n < D ? dk : dv;
    const int col = n < D ? n : n - D;
    if (dst != nullptr && column.n_ok) {
#pragma unroll
      for (int ur = 0; ur < 16 * U; ++ur) {
        const int64_t t = t0 + column.row0 + column.row_of(ur / 16, ur % 16);
        if (t < total) dst[(t * Hkv + h) * D + col] = from_f32<T>(acc[ur / 16][ur % 16]);
      }
    }
  }
}

// Forward of the first layer on bf16 storage: pre = bias + sum_tap sum_m x[t + off(tap)][m] * W[c][m][tap] with x the
// token's key and value features.  Both operands are bf16 values, so their products are exact in fp32 and the bf16
// matrix instruction (v_mfma_f32_32x32x16_bf16, fp32 accumulation) gives what the fp32 one would at 16 times the rate.
// Same tiling as conv_product_kernel: TMC tokens x TN outputs per workgroup, slices of KCB channels (a slice lies in
// the keys or in the values), the rows of a group of taps staged once; rows are read straight from k / v.
constexpr int KCB = 32, RSQ = KCB + 8;     // channels per slice; LDS row stride in elements (16-byte reads of 16 lanes
                                           // then cover all banks)
constexpr int PQA = A_ROWS * (KCB / 8) / 256, PQB = GT * TN * (KCB / 8) / 256;
static_assert(A_ROWS * (KCB / 8) % 256 == 0 && GT * TN * (KCB / 8) % 256 == 0, "whole 16-byte pieces per thread");

template <bool NARROW>
__global__ void __launch_bounds__(256, 4)
conv_first_bf16_kernel(const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int64_t stride_tok, int64_t stride_head,
                       const bf16_t* __restrict__ wq, int D, int N, int ks, int dil, const int32_t* __restrict__ seq_lo,
                       const int32_t* __restrict__ seq_hi, int64_t total, const float* __restrict__ bias,
                       float* __restrict__ pre, float* __restrict__ act, int Hkv, const OutProj<bf16_t> proj) {
  __shared__ __align__(16) bf16_t a_s[A_ROWS][RSQ];       // [staged token row][channel of the slice]
  __shared__ __align__(16) bf16_t b_s[GT][TN][RSQ];       // [tap of the group][output][channel of the slice]
  const int K = 2 * D;
  const int h = blockIdx.z;
  const int64_t t0 = (int64_t)blockIdx.x * TMC;
  const int n0 = blockIdx.y * TN;
  const int tid = threadIdx.x;
  const bf16_t* w_h = wq + (int64_t)h * ks * N * K;
  const int half = (ks - 1) / 2;
  const int lane = tid & 63, wv = tid >> 6, ql = lane & 31, hb = lane >> 5;
  constexpr int U = NARROW ? 1 : 2;                       // wave roles as in conv_product_kernel
  const int row0 = NARROW ? 32 * wv : 64 * (wv >> 1), col0 = NARROW ? 0 : 32 * (wv & 1);
  int tok32[U], lo[U], hi[U];      // token indices fit: the sequence bounds are int32
#pragma unroll
  for (int u = 0; u < U; ++u) {
    tok32[u] = (int)t0 + row0 + 32 * u + ql;
    const bool ok = tok32[u] < total;
    lo[u] = ok ? seq_lo[tok32[u]] : 0;
    hi[u] = ok ? seq_hi[tok32[u]] : 0;
  }
  f32x16 acc[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[u][r] = 0.f;
  const int per_group = min(GT, 1 + HALO / dil);
  // Staged rows outside the array and columns past N hold values of other rows or zero: what is read of them is masked below
  // with the sequence's bounds, or belongs to a column that is not written.  Rows past those that the group's taps reach are
  // not read and all take the last one's line.
  int64_t row_at[PQA];           // of the group's rows that the thread moves: element offset, clamped into the array
  uint32_t w_at[PQB];            // of its weight pieces: byte offset from the group's first tap
#pragma unroll
  for (int i = 0; i < PQB; ++i) {
    const int e = tid + 256 * i, jn = e / (KCB / 8), q = e % (KCB / 8);
    w_at[i] = (((uint32_t)(jn / TN) * (uint32_t)N + jn % TN) * (uint32_t)K + 8 * q) * 2u;
  }
  u32x4 ra[PQA], rb[PQB];
  auto fetch = [&](int tap0, int ntap, int k0) {
    if (k0 == 0) {
      const int first = (int)t0 + (tap0 - half) * dil, last = min(first + TMC - 1 + (ntap - 1) * dil, (int)total - 1);
#pragma unroll
      for (int i = 0; i < PQA; ++i) {
        const int e = tid + 256 * i;
        row_at[i] = max(0, min(first + e / (KCB / 8), last)) * stride_tok + 8 * (e % (KCB / 8));
      }
    }
    const bf16_t* src = (k0 < D ? k + k0 : v + (k0 - D)) + (int64_t)h * stride_head;      // D is a multiple of KCB
#pragma unroll
    for (int i = 0; i < PQA; ++i) ra[i] = *reinterpret_cast<const u32x4*>(src + row_at[i]);
    const auto rs_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(w_h) + ((int64_t)tap0 * N + n0) * K + k0, 0,
                                                        (((uint32_t)ntap * N - n0) * (uint32_t)K - k0) * 2u, 0x00020000);
#pragma unroll
    for (int i = 0; i < PQB; ++i) rb[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, w_at[i], 0, 0);
  };
  auto masked_piece = [](u32x4 x, bool keep) { return keep ? x : u32x4{0u, 0u, 0u, 0u}; };
  int tap0 = 0, ntap = min(per_group, ks), k0 = 0;
  fetch(tap0, ntap, k0);
  while (tap0 < ks) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PQA; ++i) {
      const int e = tid + 256 * i;
      *reinterpret_cast<u32x4*>(&a_s[e / (KCB / 8)][8 * (e % (KCB / 8))]) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < PQB; ++i) {
      const int e = tid + 256 * i, jn = e / (KCB / 8);
      *reinterpret_cast<u32x4*>(&b_s[jn / TN][jn % TN][8 * (e % (KCB / 8))]) = rb[i];
    }
    __syncthreads();
    const int tap_at = tap0, n_taps = ntap;
    k0 += KCB;
    if (k0 == K) { k0 = 0; tap0 += per_group; ntap = min(per_group, ks - tap0); }
    if (tap0 < ks) fetch(tap0, ntap, k0);
    for (int j = 0; j < n_taps; ++j) {
      const int off = (tap_at + j - half) * dil;
      const int shift = j * dil;
      bool valid[U], inside[U];      // inside: the same for all tokens of the sub-tile (no sequence ends under it)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        valid[u] = tok32[u] + off >= lo[u] && tok32[u] + off < hi[u];
        inside[u] = __builtin_amdgcn_ballot_w64(!valid[u]) == 0ull;
      }
      // lane half hb supplies channels 16 s + 8 hb .. + 7 of its row (tokens) / column (outputs) to step s
#pragma unroll
      for (int sk = 0; sk < KCB / 16; ++sk) {
        u32x4 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = *reinterpret_cast<const u32x4*>(&a_s[row0 + 32 * u + ql + shift][16 * sk + 8 * hb]);
        const u32x4 b = *reinterpret_cast<const u32x4*>(&b_s[j][col0 + ql][16 * sk + 8 * hb]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (!inside[u]) a[u] = masked_piece(a[u], valid[u]);
          acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[u]), __builtin_bit_cast(bf16x8, b),
                                                          acc[u], 0, 0, 0);
        }
      }
    }
  }
  // accumulator register r of lane half hb: token row 8*(r/4) + 4*hb + r%4 of the sub-tile, output column ql
  const int n = n0 + col0 + ql;
  const TileColumn<U> column(h, total, t0, row0 + 4 * hb, n, N);
  forward_result<U, NARROW>(proj, acc, bias, column, Hkv, pre, act, reinterpret_cast<float*>(&a_s[0][0]), wv, lane);      // one layer only: pre receives d pre
}

// x = t0 + t1 + t2 in bf16 terms (t1, t2: exact residuals), four values packed per term.  Values beyond bf16's largest would
// leave inf - inf: their first term is cut instead of rounded, and an infinity is 1 and 0 in front of itself, so that the
// products that are taken with another split value (third by first, first by third) make the infinity that the value would.
constexpr float kMaxBf16 = 3.3895314e38f;
__device__ __forceinline__ void split_quad(float4 x, uint2 (&t)[3]) {
  const float xs[4] = {x.x, x.y, x.z, x.w};
  auto pair = [](float lo, float hi) { return __builtin_bit_cast(uint32_t, bf16x2{from_f32<bf16_t>(lo), from_f32<bf16_t>(hi)}); };
  auto low = [](uint32_t p) { return __uint_as_float(p << 16); };
  auto high = [](uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); };
  float r[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    t[m] = make_uint2(pair(r[0], r[1]), pair(r[2], r[3]));
    r[0] -= low(t[m].x); r[1] -= high(t[m].x);
    r[2] -= low(t[m].y); r[3] -= high(t[m].y);
  }
  if (fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w))) > kMaxBf16) {
    auto bits = [](float y) { return (uint32_t)__builtin_bit_cast(uint16_t, from_f32<bf16_t>(y)); };
    uint32_t b[3][4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int m = 0; m < 3; ++m) b[m][c] = ((c < 2 ? t[m].x : t[m].y) >> (16 * (c % 2))) & 0xFFFFu;
      if (!(fabsf(xs[c]) > kMaxBf16)) continue;
      const bool infinite = fabsf(xs[c]) == INFINITY;
      const float top = __uint_as_float(__float_as_uint(xs[c]) & 0xFFFF0000u);
      b[0][c] = infinite ? bits(copysignf(1.f, xs[c])) : bits(top);
      b[1][c] = infinite ? 0u : bits(xs[c] - top);
      b[2][c] = infinite ? bits(xs[c]) : bits((xs[c] - top) - __uint_as_float(bits(xs[c] - top) << 16));
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) t[m] = make_uint2(b[m][0] | b[m][1] << 16, b[m][2] | b[m][3] << 16);
  }
}

// The convs whose activations are fp32 on bf16 storage: out[t][n] = sum_tap sum_k in[t + sign * off(tap)][k] * W(tap, k, n),
// sign = -1 towards the input, +1 the forward of the layers after the first.  The weights (w: [h][tap][n][k]) are bf16
// values; the fp32 operand is split into three bf16 terms (x = hi + mid + lo up to 2^-24 of x), whose products with the
// weights are exact in fp32, so three bf16 matrix instructions give the fp32 product at about five times the fp32
// instruction's rate.  Tiling as conv_product_kernel, slices of KCS channels; used when K and N are multiples of 8.
// Modes as conv_product_kernel.
constexpr int KCS = 16, RSS = KCS + 8;     // channels per slice; LDS row stride in elements
constexpr int PSA = A_ROWS * (KCS / 4) / 256, PSB = (GT * TN * (KCS / 8) + 255) / 256;
static_assert(A_ROWS * (KCS / 4) % 256 == 0, "whole quads per thread");

template <bool NARROW>
__global__ void __launch_bounds__(256, 4)
conv_split_bf16_kernel(const float* __restrict__ in, const bf16_t* __restrict__ w, int K, int N, int ks, int dil, int sign,
                       const int32_t* __restrict__ seq_lo, const int32_t* __restrict__ seq_hi, int64_t total, int Hkv,
                       int mode, const float* __restrict__ bias, const float* __restrict__ pre_prev, float* __restrict__ out0,
                       float* __restrict__ out1, bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int D,
                       const OutProj<bf16_t> proj, float* __restrict__ part_b) {
  __shared__ __align__(16) bf16_t a_s[3][A_ROWS][RSS];    // [term of the split][staged token row][channel of the slice]
  __shared__ __align__(16) bf16_t b_s[GT][TN][RSS];       // [tap of the group][output][channel of the slice]
  const int h = blockIdx.z;
  const int64_t t0 = (int64_t)blockIdx.x * TMC;
  const int n0 = blockIdx.y * TN;
  const int tid = threadIdx.x;
  const float* in_h = in + (int64_t)h * total * K;
  const bf16_t* w_h = w + (int64_t)h * ks * N * K;
  const int half = (ks - 1) / 2;
  const int lane = tid & 63, wv = tid >> 6, ql = lane & 31, hb = lane >> 5;
  constexpr int U = NARROW ? 1 : 2;                       // wave roles as in conv_product_kernel
  const int row0 = NARROW ? 32 * wv : 64 * (wv >> 1), col0 = NARROW ? 0 : 32 * (wv & 1);
  int tok32[U], lo[U], hi[U];      // token indices fit: the sequence bounds are int32
#pragma unroll
  for (int u = 0; u < U; ++u) {
    tok32[u] = (int)t0 + row0 + 32 * u + ql;
    const bool ok = tok32[u] < total;
    lo[u] = ok ? seq_lo[tok32[u]] : 0;
    hi[u] = ok ? seq_hi[tok32[u]] : 0;
  }
  f32x16 acc[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[u][r] = 0.f;
  const int per_group = min(GT, 1 + HALO / dil);
  constexpr uint32_t kOutside = 0xFFFFFFF0u;
  // Staged rows outside the array are zero, those past what the group's taps reach and columns past N hold anything: what is
  // read of them is masked below with the sequence's bounds, or belongs to a column that is not written.  Channels past K are
  // zero in both operands.
  const int qa = 4 * (tid % (KCS / 4)), qb = 8 * (tid % (KCS / 8));
  uint32_t w_at[PSB];            // of the thread's weight pieces: byte offset from the group's first tap
#pragma unroll
  for (int i = 0; i < PSB; ++i) {
    const int jn = (tid + 256 * i) / (KCS / 8);
    w_at[i] = (((uint32_t)(jn / TN) * (uint32_t)N + jn % TN) * (uint32_t)K + qb) * 2u;
  }
  u32x4 ra[PSA], rb[PSB];
  auto first_row = [&](int tap0, int ntap) { return sign > 0 ? (tap0 - half) * dil : -(tap0 + ntap - 1 - half) * dil; };
  auto fetch = [&](int tap0, int ntap, int k0) {
    const int first = (int)t0 + first_row(tap0, ntap), skip = max(0, -first);        // staged rows in front of the array
    const int rows = max(0, min(TMC + (ntap - 1) * dil, (int)total - first) - skip);
    // K % 8 == 0: whole pieces.  A row in front of the array has an offset below zero, i.e. far past the end.
    const auto rs_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(in_h) + (int64_t)(first + skip) * K + k0, 0,
                                                        rows > 0 ? ((uint32_t)rows * (uint32_t)K - k0) * 4u : 0u, 0x00020000);
#pragma unroll
    for (int i = 0; i < PSA; ++i) {
      const uint32_t at = (uint32_t)((tid / (KCS / 4) - skip + 256 / (KCS / 4) * i) * K + qa) * 4u;
      ra[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_a, k0 + qa < K ? at : kOutside, 0, 0);
    }
    const auto rs_w = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(w_h) + ((int64_t)tap0 * N + n0) * K + k0, 0,
                                                        (((uint32_t)ntap * N - n0) * (uint32_t)K - k0) * 2u, 0x00020000);
#pragma unroll
    for (int i = 0; i < PSB; ++i) rb[i] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, k0 + qb < K ? w_at[i] : kOutside, 0, 0);
  };
  auto masked_piece = [](u32x4 x, bool keep) { return keep ? x : u32x4{0u, 0u, 0u, 0u}; };
  int tap0 = 0, ntap = min(per_group, ks), k0 = 0;
  fetch(tap0, ntap, k0);
  while (tap0 < ks) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PSA; ++i) {
      const int e = tid + 256 * i, row = e / (KCS / 4), q = e % (KCS / 4);
      uint2 t[3];
      split_quad(__builtin_bit_cast(float4, ra[i]), t);
#pragma unroll
      for (int m = 0; m < 3; ++m) *reinterpret_cast<uint2*>(&a_s[m][row][4 * q]) = t[m];
    }
#pragma unroll
    for (int i = 0; i < PSB; ++i) {
      const int e = tid + 256 * i, jn = e / (KCS / 8);
      if (e < GT * TN * (KCS / 8)) *reinterpret_cast<u32x4*>(&b_s[jn / TN][jn % TN][8 * (e % (KCS / 8))]) = rb[i];
    }
    __syncthreads();
    const int tap_at = tap0, n_taps = ntap, base_off = first_row(tap0, ntap);
    k0 += KCS;
    if (k0 >= K) { k0 = 0; tap0 += per_group; ntap = min(per_group, ks - tap0); }
    if (tap0 < ks) fetch(tap0, ntap, k0);
    for (int j = 0; j < n_taps; ++j) {
      const int off = sign * (tap_at + j - half) * dil;
      const int shift = off - base_off;
      bool valid[U], inside[U];      // inside: the same for all tokens of the sub-tile (no sequence ends under it)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        valid[u] = tok32[u] + off >= lo[u] && tok32[u] + off < hi[u];
        inside[u] = __builtin_amdgcn_ballot_w64(!valid[u]) == 0ull;
      }
      // lane half hb supplies channels 8 hb .. 8 hb + 7 of its row (tokens) / column (outputs)
      u32x4 a[3][U];
#pragma unroll
      for (int m = 0; m < 3; ++m)
#pragma unroll
        for (int u = 0; u < U; ++u) a[m][u] = *reinterpret_cast<const u32x4*>(&a_s[m][row0 + 32 * u + ql + shift][8 * hb]);
      const u32x4 b = *reinterpret_cast<const u32x4*>(&b_s[j][col0 + ql][8 * hb]);
#pragma unroll
      for (int m = 2; m >= 0; --m)        // smallest terms first
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (!inside[u]) a[m][u] = masked_piece(a[m][u], valid[u]);
          acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[m][u]), __builtin_bit_cast(bf16x8, b),
                                                          acc[u], 0, 0, 0);
        }
    }
  }
  // accumulator register r of lane half hb: token row 8*(r/4) + 4*hb + r%4 of the sub-tile, output column ql
  const int n = n0 + col0 + ql;
  const TileColumn<U> column(h, total, t0, row0 + 4 * hb, n, N);
  if (mode == 0) {
    forward_result<U, NARROW>(proj, acc, bias, column, Hkv, out0, out1, reinterpret_cast<float*>(&a_s[0][0][0]), wv, lane);
  } else if (mode == 1) {
    hidden_backward<U, NARROW>(acc, column, Hkv, pre_prev, out0, part_b, reinterpret_cast<float*>(&a_s[0][0][0]), wv, lane);
  } else {
    // N = 2 D and D is a multiple of TN: the workgroup's columns are all keys' or all values'
    bf16_t* const dst = n0 < D ? dk : dv;
    const int first = n0 < D ? n0 : n0 - D;
    if (dst != nullptr && !NARROW) {      // rows through LDS, 16 bytes per lane
      constexpr int RSO = TN + 8;
      static_assert(sizeof(a_s) >= TMC * RSO * sizeof(bf16_t), "the tile fits the staging rows");
      bf16_t* const o_s = &a_s[0][0][0];
      __syncthreads();
#pragma unroll
      for (int ur = 0; ur < 16 * U; ++ur)
        o_s[(row0 + 32 * (ur / 16) + 8 * ((ur % 16) / 4) + 4 * hb + (ur % 4)) * RSO + col0 + ql] = from_f32<bf16_t>(acc[ur / 16][ur % 16]);
      __syncthreads();
      const int rows_left = (int)(total - t0 < TMC ? total - t0 : TMC);
      bf16_t* const o_t = dst + (t0 * Hkv + h) * D + first;
#pragma unroll
      for (int i = 0; i < TMC * (TN / 8) / 256; ++i) {
        const int e = tid + 256 * i, row = e / (TN / 8), q = e % (TN / 8);
        if (row < rows_left)
          *reinterpret_cast<u32x4*>(o_t + (int64_t)row * Hkv * D + 8 * q) = *reinterpret_cast<const u32x4*>(o_s + row * RSO + 8 * q);
      }
    }
  }
}

// Stage 1 of d W_l: partial[chunk][h][tap][c][m] = sum over the chunk's tokens t of a_{l-1}[t + off][m] * d y_l[t][c],
// a tiled fp32 product with the tokens as the contraction index (slices of KCW tokens through LDS).  The chunk's
// sequence bounds are staged in LDS first, so a slice's operands need one round of global loads, not two dependent
// ones; the output channels are the rows of the matrix tiles, so neighbouring lanes write neighbouring m.
template <int WC, int WM>
__global__ void __launch_bounds__(256)
weight_product_kernel(const float* __restrict__ act_in, const float* __restrict__ dpre, int Cin, int Cout, int ks, int dil,
                      const int32_t* __restrict__ seq_lo, const int32_t* __restrict__ seq_hi, int64_t total, int Hkv,
                      int tiles_n, int tiles, int n_work, int chunk_tokens, float* __restrict__ partial) {
  // [operand][token of the slice][channel ^ 32 * (token & 1)]: the two lane halves of an operand read take neighbouring
  // tokens, and the swap of the row halves on odd tokens puts them on different banks without padding the rows
  __shared__ float ab_s[2][KCW][64];
  float (*a_s)[64] = ab_s[0];          // activations, channel = m
  float (*b_s)[64] = ab_s[1];          // d y, channel = c
  __shared__ int32_t lo_s[kTokChunk], hi_s[kTokChunk];
  // Workgroups are dealt round-robin to the 8 XCDs; each XCD gets a contiguous range of work items, ordered (tile,
  // tap, head, chunk), so that the tiles and taps of one (head, chunk), which read the same rows, meet in one L2.
  const int per_xcd = (n_work + 7) / 8;
  const int work = ((int)blockIdx.x % 8) * per_xcd + (int)blockIdx.x / 8;
  if (work >= n_work) return;
  const int tile = work % tiles, head_tap = (work / tiles) % (Hkv * ks);
  const int m0 = (tile / tiles_n) * (32 * WM), c0 = (tile % tiles_n) * (32 * WC);
  const int h = head_tap / ks, tap = head_tap % ks;
  const int chunk = work / (tiles * Hkv * ks);
  const int tid = threadIdx.x;
  const int off = (tap - (ks - 1) / 2) * dil;
  const int64_t tb = (int64_t)chunk * chunk_tokens;
  const int64_t te = tb + chunk_tokens < total ? tb + chunk_tokens : total;
  const float* a_h = act_in + (int64_t)h * total * Cin;
  const float* g_h = dpre + (int64_t)h * total * Cout;
  const int lane = tid & 63, wv = tid >> 6, ql = lane & 31, hb = lane >> 5;
  // Wave roles: WC x WM waves tile the output (32 output channels x 32 input channels each); when that takes fewer than
  // four, the S waves of a tile take every S-th pair of tokens of a slice and their sums are added in wave order.
  constexpr int S = 4 / (WC * WM);
  const int wq = wv % (WC * WM), sp = wv / (WC * WM), ci = wq / WM, mi = wq % WM;
  for (int i = tid; i < chunk_tokens; i += 256) {
    const bool ok = tb + i < te;
    lo_s[i] = ok ? seq_lo[tb + i] : 0;
    hi_s[i] = ok ? seq_hi[tb + i] : 0;   // an empty range: rows past the chunk's end contribute nothing
  }
  __syncthreads();
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  // A thread moves channel x of tokens wv, wv + 4, ... of a slice.  Token indices are kept relative to the chunk, in
  // 32 bits (the token count fits: the bounds are int32), so that a load costs little address arithmetic.
  const int x = tid & 63;
  const bool m_ok = x < 32 * WM && m0 + x < Cin, c_ok = x < 32 * WC && c0 + x < Cout;
  const float* a_col = a_h + tb * Cin + min(m0 + x, Cin - 1);
  const float* g_col = g_h + tb * Cout + min(c0 + x, Cout - 1);
  const int len = (int)(te - tb), tb32 = (int)tb;
  float ra[PERW], rb[PERW];
  unsigned keep_a, keep_b;     // one bit per loaded value: does it count
  auto fetch = [&](int i0) {
    keep_a = keep_b = 0u;
#pragma unroll
    for (int j = 0; j < PERW; ++j) {
      const int i = i0 + wv + 4 * j;                 // token of the chunk
      const bool t_ok = i < len;
      const int ic = t_ok ? i : 0;
      const int p = tb32 + ic + off;
      const bool p_ok = t_ok & (p >= lo_s[ic]) & (p < hi_s[ic]);
      // unconditional loads from rows inside the arrays; what does not count is zeroed where the value is consumed
      ra[j] = a_col[(int64_t)(p_ok ? ic + off : 0) * Cin];
      rb[j] = g_col[(int64_t)ic * Cout];
      keep_a |= (p_ok && m_ok) ? 1u << j : 0u;
      keep_b |= (t_ok && c_ok) ? 1u << j : 0u;
    }
  };
  fetch(0);
  for (int i0 = 0; i0 < len; i0 += KCW) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PERW; ++j) {
      a_s[wv + 4 * j][x ^ ((wv & 1) << 5)] = masked_value(ra[j], keep_a >> j & 1u);      // token parity = wv & 1
      b_s[wv + 4 * j][x ^ ((wv & 1) << 5)] = masked_value(rb[j], keep_b >> j & 1u);
    }
    __syncthreads();
    if (i0 + KCW < len) fetch(i0 + KCW);   // the next slice's operands travel while this one is multiplied
#pragma unroll
    for (int tt = 2 * sp; tt < KCW; tt += 2 * S)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b_s[tt + hb][(32 * ci + ql) ^ (hb << 5)],
                                                 a_s[tt + hb][(32 * mi + ql) ^ (hb << 5)], acc, 0, 0, 0);   // tt is even
  }
  if constexpr (S > 1) {
    float* red = &ab_s[0][0][0];       // (S - 1) * WC * WM accumulator tiles of 1024 floats fit the operand tiles
    __syncthreads();
    if (sp > 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) red[((sp - 1) * WC * WM + wq) * 1024 + r * 64 + lane] = acc[r];
    }
    __syncthreads();
    if (sp > 0) return;
    for (int k = 1; k < S; ++k)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += red[((k - 1) * WC * WM + wq) * 1024 + r * 64 + lane];
  }
  float* out = partial + (((int64_t)chunk * Hkv + h) * ks + tap) * Cout * Cin;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int c = c0 + 32 * ci + 8 * (r / 4) + 4 * hb + (r % 4);
    const int m = m0 + 32 * mi + ql;
    if (m < Cin && c < Cout) out[(int64_t)c * Cin + m] = acc[r];
  }
}

// Stage 1 of d W_l on bf16 storage, for the channel counts that come in whole quads.  d y (fp32) is split into three bf16
// terms as in conv_split_bf16_kernel.  X = bf16_t: the first layer, whose inputs are bf16 values, so three bf16 matrix
// instructions give the fp32 product.  X = float: the layers after it; the activations are split too, and the six products of
// terms down to 2^-16 of the largest are taken (the three others are below 2^-25 of it).  Not the fp32 instruction's result to
// the last bit; relative error of the three layers' weight gradients against 64 bits (2 x 1500 tokens, paper stack): 3.3e-7,
// 3.6e-7 and 3.6e-7 on fp32 instructions, 2.4e-7, 2.6e-7 and 2.6e-7 in this form.
// A workgroup takes one (head, chunk of tokens, tile of 32 WM input x 32 WC output channels) and a group of taps: d y is
// loaded and split once for all of them, and the input rows that the taps reach are staged once and read at each tap's shift.
// (A workgroup per tap spent its time on loading and splitting the same rows: 4 x 4096 tokens, paper stack, 49 us for the
// first layer and, on fp32 instructions, 43 and 35 for the next two; 16 heads of D = 128, k = 5: 234 us.)
// The contraction runs over the tokens, i.e. over the rows of the staged [token][channel] tiles: both operands are fetched
// with transposing LDS loads (eight consecutive tokens of one channel per lane); the row strides put four consecutive rows'
// 64 bytes on different banks.  Whether a tap's row lies in the token's own sequence: one bit per token of a slice in a
// scalar mask, applied to the operand where any bit is clear.  Waves: WC x WM of them tile the output; where that takes fewer
// than four, the S waves of a block take every S-th step of tokens and their sums are added in wave order.
constexpr int KCT = 64, NTW = 4;             // tokens per slice; most taps per group
template <class X, int WC, int WM> struct WeightTile {
  static constexpr bool kSplit = std::is_same<X, float>::value;
  static constexpr int S = 4 / (WC * WM), MT = 32 * WM, CT = 32 * WC, XT = kSplit ? 3 : 1;
  static constexpr int kHalo = kSplit ? 16 : 64, XR = KCT + kHalo;
  static constexpr int RSX = MT == 32 ? 32 : MT + 32, RSG = CT == 32 ? 32 : CT + 32;     // row strides in elements
  static constexpr int EPX = kSplit ? 4 : 8;                                             // channels per loaded piece
  static constexpr int PX = (XR * (MT / EPX) + 255) / 256, PG = KCT * (CT / 4) / 256;
  static constexpr int kXElems = XT * XR * RSX, kElems = kXElems + 3 * KCT * RSG;
  static_assert(kElems * 2 >= (S - 1) * WC * WM * 4096, "the waves' sums are exchanged in the tiles");
};
// Taps per group and groups, balanced.
inline int weight_groups(int ks, int dil, bool split) {
  const int reach = 1 + (split ? 16 : 64) / dil, most = reach < NTW ? reach : NTW;
  return (ks + most - 1) / most;
}

// Input channel m is x0's for m < split, else x1's channel m - split (the keys and the values; one array for X = float).
// <float, 2, 1> runs two waves per SIMD: 30.1 and 56.1 us (4 x 4096 tokens, 8 heads, a k = 3 layer of 32 -> 64 and a k = 5 layer of
// 32 -> 128 channels); held to the registers of three 31.9 and 58.8.
template <class X, int WC, int WM>
__global__ void __launch_bounds__(256)
weight_split_kernel(const X* __restrict__ x0, const X* __restrict__ x1, int split, int64_t stride_tok, int64_t stride_head,
                    const float* __restrict__ dpre, int Cin, int Cout, int ks, int dil, const int32_t* __restrict__ seq_lo,
                    const int32_t* __restrict__ seq_hi, int64_t total, int Hkv, int tiles_n, int tiles, int groups, int n_work,
                    int chunk_tokens, float* __restrict__ partial) {
  using G = WeightTile<X, WC, WM>;
  constexpr int S = G::S, MT = G::MT, CT = G::CT, RSX = G::RSX, RSG = G::RSG, EPX = G::EPX, XQ = MT / EPX, GQ = CT / 4;
  __shared__ __align__(16) bf16_t lds[G::kElems];
  bf16_t* const x_s = lds;                  // [term][staged row][channel]
  bf16_t* const g_s = lds + G::kXElems;     // [term][token of the slice][channel]
  // XCD-contiguous work order (tile, group, head, chunk): the tiles of one (head, chunk) read the same rows
  const int per_xcd = (n_work + 7) / 8;
  const int work = ((int)blockIdx.x % 8) * per_xcd + (int)blockIdx.x / 8;
  if (work >= n_work) return;
  const int tile = work % tiles, head_group = (work / tiles) % (Hkv * groups);
  const int m0 = (tile / tiles_n) * MT, c0 = (tile % tiles_n) * CT;
  const int h = head_group / groups;
  const int chunk = work / (tiles * Hkv * groups);
  const int per = (ks + groups - 1) / groups, tap0 = (head_group % groups) * per, ntap = min(per, ks - tap0);
  const int off0 = (tap0 - (ks - 1) / 2) * dil;
  const int tid = threadIdx.x, lane = tid & 63, hb = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq = wv % (WC * WM), sp = wv / (WC * WM), ci = wq / WM, mi = wq % WM;
  const int64_t tb = (int64_t)chunk * chunk_tokens;
  const int64_t te = tb + chunk_tokens < total ? tb + chunk_tokens : total;
  const int len = (int)(te - tb), tb32 = (int)tb, total32 = (int)total;
  const float* g_h = dpre + ((int64_t)h * total + tb) * Cout;
  const X* x0_h = x0 + (int64_t)h * stride_head;
  const X* x1_h = x1 + (int64_t)h * stride_head;

  f32x16 acc[NTW];
#pragma unroll
  for (int j = 0; j < NTW; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  u32x4 rx[G::PX], rg[G::PG];
  int lo, hi;                    // bounds of the sequence of the slice's token `lane`; empty past the chunk
  // Rows of d y past the chunk are zero.  Input rows outside the array and channels past Cin or Cout hold anything: the
  // sequence's bounds mask them below, or they belong to a sum that is not written.  Rows past those that the taps reach are
  // not read and all take the last one's line.
  static_assert(256 % XQ == 0 && 256 % GQ == 0, "a thread keeps its channels");
  const int mc = min(m0 + EPX * (tid % XQ), Cin - EPX);
  const X* const x_col = mc < split ? x0_h + mc : x1_h + (mc - split);
  const uint32_t g_at = ((uint32_t)(tid / GQ) * (uint32_t)Cout + 4 * (tid % GQ)) * 4u;
  auto fetch = [&](int i0) {
    const int first = tb32 + i0 + off0, last = min(first + KCT - 1 + (ntap - 1) * dil, total32 - 1);
#pragma unroll
    for (int j = 0; j < G::PX; ++j)
      rx[j] = *reinterpret_cast<const u32x4*>(x_col + max(0, min(first + tid / XQ + 256 / XQ * j, last)) * stride_tok);
    const auto rs_g = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g_h) + (int64_t)i0 * Cout + c0, 0,
                                                        ((uint32_t)min(KCT, len - i0) * (uint32_t)Cout - c0) * 4u, 0x00020000);
#pragma unroll
    for (int j = 0; j < G::PG; ++j)
      rg[j] = __builtin_amdgcn_raw_buffer_load_b128(rs_g, g_at + (uint32_t)(256 / GQ * j) * (uint32_t)Cout * 4u, 0, 0);
    const int t = i0 + lane < len ? tb32 + i0 + lane : tb32;
    lo = seq_lo[t];
    hi = seq_hi[t];
    if (i0 + lane >= len) hi = lo;
  };
  // transposing loads: in each group of 16 lanes, lane j points at row j / 4, columns 4 * (j % 4) .. of its 16 columns
  const int tr_row = 8 * hb + ((lane & 15) >> 2), tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const bf16_t* const g_op = g_s + tr_row * RSG + 32 * ci + tr_col;
  const bf16_t* const x_op = x_s + tr_row * RSX + 32 * mi + tr_col;
  fetch(0);
  for (int i0 = 0; i0 < len; i0 += KCT) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < G::PX; ++j) {
      const int e = tid + 256 * j;
      const u32x4 x = rx[j];
      bf16_t* dst = x_s + (e / XQ) * RSX + EPX * (e % XQ);
      if (e < G::XR * XQ) {
        if constexpr (G::kSplit) {
          uint2 t[3];
          split_quad(__builtin_bit_cast(float4, x), t);
#pragma unroll
          for (int m = 0; m < 3; ++m) *reinterpret_cast<uint2*>(dst + m * G::XR * RSX) = t[m];
        } else {
          *reinterpret_cast<u32x4*>(dst) = x;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < G::PG; ++j) {
      const int e = tid + 256 * j;
      uint2 t[3];
      split_quad(__builtin_bit_cast(float4, rg[j]), t);
#pragma unroll
      for (int m = 0; m < 3; ++m) *reinterpret_cast<uint2*>(g_s + (m * KCT + e / GQ) * RSG + 4 * (e % GQ)) = t[m];
    }
    uint64_t valid[NTW];           // bit i: token i of the slice has a row of its own sequence under the tap
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
      const int p = tb32 + i0 + lane + off0 + j * dil;
      valid[j] = __builtin_amdgcn_ballot_w64(p >= lo && p < hi);
    }
    __syncthreads();
    if (i0 + KCT < len) fetch(i0 + KCT);
#pragma unroll
    for (int st = sp; st < KCT / 16; st += S) {              // steps of 16 tokens
      bf16x8 a[3];
#pragma unroll
      for (int m = 0; m < 3; ++m) a[m] = load_transposed(g_op + (m * KCT + 16 * st) * RSG, RSG);
#pragma unroll
      for (int j = 0; j < NTW; ++j) {
        if (j >= ntap) break;
        bf16x8 b[G::XT];
#pragma unroll
        for (int m = 0; m < G::XT; ++m) b[m] = load_transposed(x_op + (m * G::XR + 16 * st + j * dil) * RSX, RSX);
        if (valid[j] != ~0ull) {
          const uint32_t bits = (uint32_t)(valid[j] >> (16 * st)) >> (8 * hb);
#pragma unroll
          for (int m = 0; m < G::XT; ++m) {
            u32x4 w = __builtin_bit_cast(u32x4, b[m]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              w[i] &= ((bits >> (2 * i) & 1u) ? 0xFFFFu : 0u) | ((bits >> (2 * i + 1) & 1u) ? 0xFFFF0000u : 0u);
            b[m] = __builtin_bit_cast(bf16x8, w);
          }
        }
        // smallest terms first
        if constexpr (G::kSplit) {
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc[j], 0, 0, 0);
        } else {
#pragma unroll
          for (int m = 2; m >= 0; --m) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m], b[0], acc[j], 0, 0, 0);
        }
      }
    }
  }
  float* out = partial + (((int64_t)chunk * Hkv + h) * ks + tap0) * Cout * Cin;
  const int m = m0 + 32 * mi + (lane & 31), first_c = c0 + 32 * ci;
#pragma unroll
  for (int j = 0; j < NTW; ++j) {
    if (j >= ntap) break;
    if constexpr (S > 1) {
      float* red = reinterpret_cast<float*>(lds);       // (S - 1) * WC * WM accumulator tiles of 1024 floats
      __syncthreads();
      if (sp > 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) red[((sp - 1) * WC * WM + wq) * 1024 + r * 64 + lane] = acc[j][r];
      }
      __syncthreads();
      if (sp == 0) {
        for (int k = 1; k < S; ++k)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[j][r] += red[((k - 1) * WC * WM + wq) * 1024 + r * 64 + lane];
      }
    }
    // a 64-bit row address in scalar registers, the lane's 32 bits beside it
    if (sp == 0 && m < Cin) {
      float* const out_j = out + (int64_t)j * Cout * Cin;
      const uint32_t at = (uint32_t)(4 * hb) * (uint32_t)Cin + m;
      auto store = [&](bool whole) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = 8 * (r / 4) + r % 4;
          if (whole || first_c + 4 * hb + row < Cout) (out_j + (int64_t)(first_c + row) * Cin)[at] = acc[j][r];
        }
      };
      if (first_c + 32 <= Cout) store(true);
      else store(false);
    }
  }
}

// Stage 2: out[i] = sum over chunks of partial[chunk][i], in chunk order.
__global__ void __launch_bounds__(256)
chunk_sum_kernel(const float* __restrict__ partial, int64_t n, int chunks, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float acc = 0.f;
#pragma unroll 8
  for (int ch = 0; ch < chunks; ++ch) acc += partial[(int64_t)ch * n + i];
  out[i] = acc;
}

// Stage 2 of every sum of a call in one launch: blockIdx.y picks the sum, its elements summed over the chunks in chunk order.
// A weight sum's partials come as [head][tap][c][m], rows of which the workgroups write whole, and go out as [head][c][m][tap]:
// per is C_l * C_{l-1} there (taps 1: in the order that they come in).  (Partials in the weights' own order, each line written
// once per tap in pieces of 4 bytes: first layer's weight product 34.1 us, this way 32.0; 4 x 4096 tokens, paper stack.)
constexpr int kMaxSums = 2 * LTEA_MAX_CNN_LAYERS + 2;
struct SumSeg { const float* partial; float* out; int64_t n; int chunks, taps; int64_t per; };
struct SumSegs { SumSeg s[kMaxSums]; };
__global__ void __launch_bounds__(256)
chunk_sum_all_kernel(const SumSegs S) {
  const SumSeg seg = S.s[blockIdx.y];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= seg.n) return;
  float acc = 0.f;
#pragma unroll 8
  for (int ch = 0; ch < seg.chunks; ++ch) acc += seg.partial[(int64_t)ch * seg.n + i];
  int64_t o = i;
  if (seg.taps > 1) {
    int64_t block, in_block;       // of [head][tap], and the element in it
    if (seg.n >> 32) { block = i / seg.per; in_block = i - block * seg.per; }
    else { block = (uint32_t)i / (uint32_t)seg.per; in_block = (uint32_t)i - (uint32_t)block * (uint32_t)seg.per; }
    const uint32_t head = (uint32_t)block / (uint32_t)seg.taps, tap = (uint32_t)block - head * (uint32_t)seg.taps;
    o = (head * seg.per + in_block) * seg.taps + tap;
  }
  seg.out[o] = acc;
}

// How a layer's weight product is cut: channel blocks per tile, tiles, tap groups and tokens per partial.
struct WeightPlan { bool split; int wc, wm, tiles_n, tiles, groups, chunk, chunks; };
WeightPlan weight_plan(const ltea_cfg& cfg, const ltea_cnn& cnn, int l, int64_t total) {
  const int cin = l == 0 ? 2 * cfg.D : cnn.c_out[l - 1], cout = cnn.c_out[l], ks = cnn.kernel[l];
  WeightPlan P;
  P.split = cfg.dtype == LTEA_BF16 && cin % 4 == 0 && cout % 4 == 0;      // whole quads
  // 32-wide halves of the 64 x 64 tile that a narrow layer would leave empty go to sharing the tokens instead, or (the
  // first layer's inputs, 2 D >= 128 channels) to a tile of 128 input channels
  P.wc = cout <= 32 ? 1 : 2;
  P.wm = P.split && l == 0 ? 4 / P.wc : (cin <= 32 ? 1 : 2);
  P.tiles_n = (cout + 32 * P.wc - 1) / (32 * P.wc);
  P.tiles = ((cin + 32 * P.wm - 1) / (32 * P.wm)) * P.tiles_n;
  P.groups = P.split ? weight_groups(ks, cnn.dilation[l], l > 0) : ks;
  // A workgroup walks its chunk slice by slice, a memory round trip each, so a launch is as long as a chunk until the chip is
  // full: chunks are halved while fewer than 512 workgroups (two per CU) would run.  Not below 128 tokens: a partial is as
  // large as the weights, and each is written and read once.
  P.chunk = kTokChunk;
  while (P.chunk > 128 && (int64_t)P.tiles * cfg.Hkv * P.groups * ((total + P.chunk - 1) / P.chunk) < 512) P.chunk /= 2;
  P.chunks = (int)((total + P.chunk - 1) / P.chunk);
  return P;
}
// The most partials that any total up to this one takes (a shorter one may be cut finer): with W workgroups per partial and
// n = ceil(512 / W), fewer than n chunks are halved, so a finer cut never exceeds 2 (n - 1) of them.
int64_t most_chunks(const ltea_cfg& cfg, const ltea_cnn& cnn, int l, int64_t total) {
  const WeightPlan P = weight_plan(cfg, cnn, l, total);
  const int64_t w = (int64_t)P.tiles * cfg.Hkv * P.groups, finer = 2 * ((512 + w - 1) / w - 1);
  const int64_t shortest = (total + 127) / 128, longest = (total + kTokChunk - 1) / kTokChunk;
  const int64_t most = shortest < finer ? shortest : finer;
  return most > longest ? most : longest;
}

size_t up256(size_t x) { return (x + 255) / 256 * 256; }

struct Layout {
  int32_t *seq_lo, *seq_hi;
  float* a0;                                  // [Hkv][T][2D] input features as fp32
  float* pre[LTEA_MAX_CNN_LAYERS];            // [Hkv][T][C_l], all but the last layer's
  float* act[LTEA_MAX_CNN_LAYERS];
  float* dpre[2];                             // [Hkv][T][widest layer], ping-pong
  float *wf[LTEA_MAX_CNN_LAYERS], *wb[LTEA_MAX_CNN_LAYERS];   // fp32 weight panels of every layer
  void* wq[LTEA_MAX_CNN_LAYERS];              // every layer's weights [Hkv][k][C_l][C_{l-1}] in the storage type (bf16 only)
  void* wqf[LTEA_MAX_CNN_LAYERS];             // every layer's weights [Hkv][k][C_{l-1}][C_l] in the storage type (bf16 only)
  float* part_w[LTEA_MAX_CNN_LAYERS];         // [chunks][Hkv][k][C_l][C_{l-1}]: partial weight gradients
  float* part_b[LTEA_MAX_CNN_LAYERS];         // [tiles of TMC tokens][Hkv][C_l]: partial bias gradients
  float *part_wout, *part_bout;               // [tiles of TMC tokens][Hkv][C_L], [tiles][Hkv]
  size_t bytes;
};

// most: room for every total up to this one (what the size query reports), else for exactly this one.
Layout carve(const ltea_cfg& cfg, const ltea_cnn& cnn, int64_t total, void* base, bool most = false) {
  Layout L;
  uintptr_t p = reinterpret_cast<uintptr_t>(base);   // integer arithmetic: a size query carves from a null base
  auto take = [&](size_t bytes) { char* r = reinterpret_cast<char*>(p); p += up256(bytes); return r; };
  const size_t rows = (size_t)cfg.Hkv * (size_t)total;
  L.seq_lo = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)total));
  L.seq_hi = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)total));
  L.a0 = reinterpret_cast<float*>(take(sizeof(float) * rows * 2 * cfg.D));
  int cmax = 0;
  int cin = 2 * cfg.D;
  for (int l = 0; l < LTEA_MAX_CNN_LAYERS; ++l) L.pre[l] = L.act[l] = nullptr;
  for (int l = 0; l < cnn.n_layers; ++l) {
    if (l < cnn.n_layers - 1) {
      L.pre[l] = reinterpret_cast<float*>(take(sizeof(float) * rows * cnn.c_out[l]));
      L.act[l] = reinterpret_cast<float*>(take(sizeof(float) * rows * cnn.c_out[l]));
    }
    cmax = cnn.c_out[l] > cmax ? cnn.c_out[l] : cmax;
    cin = cnn.c_out[l];
  }
  for (int i = 0; i < 2; ++i) L.dpre[i] = reinterpret_cast<float*>(take(sizeof(float) * rows * cmax));
  cin = 2 * cfg.D;
  for (int l = 0; l < LTEA_MAX_CNN_LAYERS; ++l) L.wf[l] = L.wb[l] = nullptr;
  for (int l = 0; l < cnn.n_layers; ++l) {
    const size_t w = (size_t)cfg.Hkv * cnn.c_out[l] * cin * cnn.kernel[l];
    L.wf[l] = reinterpret_cast<float*>(take(sizeof(float) * w));
    L.wb[l] = reinterpret_cast<float*>(take(sizeof(float) * w));
    cin = cnn.c_out[l];
  }
  cin = 2 * cfg.D;
  for (int l = 0; l < LTEA_MAX_CNN_LAYERS; ++l) L.wq[l] = L.wqf[l] = nullptr;
  for (int l = 0; l < cnn.n_layers; ++l) {
    if (cfg.dtype != LTEA_F32) {
      L.wq[l] = take(sizeof(bf16_t) * (size_t)cfg.Hkv * cnn.c_out[l] * cin * cnn.kernel[l]);
      L.wqf[l] = take(sizeof(bf16_t) * (size_t)cfg.Hkv * cnn.c_out[l] * cin * cnn.kernel[l]);
    }
    cin = cnn.c_out[l];
  }
  const size_t col_chunks = (size_t)((total + TMC - 1) / TMC);
  cin = 2 * cfg.D;
  for (int l = 0; l < LTEA_MAX_CNN_LAYERS; ++l) L.part_w[l] = L.part_b[l] = nullptr;
  for (int l = 0; l < cnn.n_layers; ++l) {
    const size_t chunks = (size_t)(most ? most_chunks(cfg, cnn, l, total) : weight_plan(cfg, cnn, l, total).chunks);
    L.part_w[l] = reinterpret_cast<float*>(take(sizeof(float) * chunks * cfg.Hkv * cnn.c_out[l] * cin * cnn.kernel[l]));
    L.part_b[l] = reinterpret_cast<float*>(take(sizeof(float) * col_chunks * cfg.Hkv * cnn.c_out[l]));
    cin = cnn.c_out[l];
  }
  L.part_wout = reinterpret_cast<float*>(take(sizeof(float) * col_chunks * cfg.Hkv * cin));
  L.part_bout = reinterpret_cast<float*>(take(sizeof(float) * col_chunks * cfg.Hkv));
  L.bytes = (size_t)(p - reinterpret_cast<uintptr_t>(base));
  return L;
}

template <typename T>
hipError_t run(const ltea_cfg& cfg, const ltea_cnn& cnn, const void* k, const void* v, int64_t stride_tok,
               int64_t stride_head, const SeqView& sv, const float* dz, const ltea_cnn_grad& g, void* dk, void* dv,
               void* workspace, hipStream_t stream) {
  const int64_t total = sv.total_tokens;
  const int Hkv = cfg.Hkv, nl = cnn.n_layers, D = cfg.D;
  const Layout L = carve(cfg, cnn, total, workspace);
  hipError_t e;
  const unsigned tok_tiles = (unsigned)((total + TMC - 1) / TMC);
  auto cin_of = [&](int l) { return l == 0 ? 2 * D : cnn.c_out[l - 1]; };
  auto in_of = [&](int l) -> const float* { return l == 0 ? L.a0 : L.act[l - 1]; };
  // rows of both operands in whole, 16-byte aligned quads: the vector-load instance
  auto conv_product = [](int K, int N) {
    const bool vec = K % 4 == 0 && N % 4 == 0;
    if (N <= 32) return vec ? conv_product_kernel<T, true, true> : conv_product_kernel<T, false, true>;
    return vec ? conv_product_kernel<T, true, false> : conv_product_kernel<T, false, false>;
  };
  // on bf16 storage, the layers whose convs take the bf16 kernels, whole 16-byte pieces of both weight orders (the first
  // layer's forward always does)
  constexpr bool kBf16 = std::is_same<T, bf16_t>::value;
  auto on_bf16 = [&](int l) { return kBf16 && cnn.c_out[l] % 8 == 0 && cin_of(l) % 8 == 0; };
  {
    PrepareArgs P;
    P.n_layers = nl; P.cu = sv.cu_seqlens; P.n_seqs = sv.n_seqs; P.total = total; P.seq_lo = L.seq_lo; P.seq_hi = L.seq_hi;
    int64_t most = total;
    for (int l = 0; l < nl; ++l) {
      const int64_t n = (int64_t)Hkv * cnn.c_out[l] * cin_of(l) * cnn.kernel[l];
      const bool fwd = on_bf16(l) || (kBf16 && l == 0), back = on_bf16(l);
      P.layer[l] = LayerPanels{cnn.w[l], fwd ? nullptr : L.wf[l], back ? nullptr : L.wb[l], fwd ? L.wq[l] : nullptr,
                               back ? L.wqf[l] : nullptr, cin_of(l), cnn.c_out[l], cnn.kernel[l], n};
      most = n > most ? n : most;
    }
    hipLaunchKernelGGL(prepare_kernel<T>, dim3((unsigned)((most + 255) / 256), (unsigned)(nl + 1)), dim3(256), 0, stream, P);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // on bf16 storage the first layer's kernels read k / v themselves, unless its weight product takes the fp32 route
  if (!weight_plan(cfg, cnn, 0, total).split) {
    hipLaunchKernelGGL(features_kernel<T>, dim3((unsigned)((total * (2 * D / Elems<T>::N) + 255) / 256), (unsigned)Hkv), dim3(256),
                       0, stream, static_cast<const T*>(k), static_cast<const T*>(v), stride_tok, stride_head, D, total, L.a0);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // 1. forward, pre-activations and activations kept; 2. the output projection, in the last layer's launch
  for (int l = 0; l < nl; ++l) {
    const int N = cnn.c_out[l];
    const bool last = l == nl - 1;
    const OutProj<T> proj = {last ? dz : nullptr, static_cast<const T*>(cnn.w_out), L.part_b[l], L.part_wout, L.part_bout};
    float* const out0 = last ? L.dpre[0] : L.pre[l];
    if constexpr (std::is_same<T, bf16_t>::value) {
      if (l == 0) {     // both operands are bf16 values: the bf16 matrix instruction gives the fp32 result
        const dim3 grid(tok_tiles, (unsigned)((N + TN - 1) / TN), (unsigned)Hkv);
        hipLaunchKernelGGL(N <= 32 ? conv_first_bf16_kernel<true> : conv_first_bf16_kernel<false>, grid, dim3(256), 0, stream,
                           static_cast<const bf16_t*>(k), static_cast<const bf16_t*>(v), stride_tok, stride_head,
                           static_cast<const bf16_t*>(L.wq[0]), D, N, cnn.kernel[0], cnn.dilation[0], L.seq_lo, L.seq_hi, total,
                           cnn.bias[0], out0, L.act[0], Hkv, proj);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        continue;
      }
      if (on_bf16(l)) {
        hipLaunchKernelGGL(N <= 32 ? conv_split_bf16_kernel<true> : conv_split_bf16_kernel<false>,
                           dim3(tok_tiles, (unsigned)((N + TN - 1) / TN), (unsigned)Hkv), dim3(256), 0, stream, in_of(l),
                           static_cast<const bf16_t*>(L.wq[l]), cin_of(l), N, cnn.kernel[l], cnn.dilation[l], 1, L.seq_lo, L.seq_hi,
                           total, Hkv, 0, cnn.bias[l], static_cast<const float*>(nullptr), out0, L.act[l],
                           static_cast<bf16_t*>(nullptr), static_cast<bf16_t*>(nullptr), D, proj, static_cast<float*>(nullptr));
        if ((e = hipGetLastError()) != hipSuccess) return e;
        continue;
      }
    }
    hipLaunchKernelGGL(conv_product(cin_of(l), N), dim3(tok_tiles, (unsigned)((N + TN - 1) / TN), (unsigned)Hkv), dim3(256), 0,
                       stream, in_of(l), L.wf[l], cin_of(l), N, cnn.kernel[l], cnn.dilation[l], 1, L.seq_lo, L.seq_hi, total,
                       Hkv, 0, cnn.bias[l], static_cast<const float*>(nullptr), out0, L.act[l], static_cast<T*>(nullptr),
                       static_cast<T*>(nullptr), D, proj, static_cast<float*>(nullptr));
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int CL = cnn.c_out[nl - 1];
  const int col_chunks = (int)((total + TMC - 1) / TMC);
  // every sum's second stage runs in one launch at the end
  SumSegs sums;
  int n_sums = 0;
  int64_t n_sum_max = 0;
  auto second_stage = [&](const float* partial, float* out, int64_t n, int n_chunks, int taps = 1, int64_t per = 0) {
    sums.s[n_sums++] = SumSeg{partial, out, n, n_chunks, taps, per};
    n_sum_max = n > n_sum_max ? n : n_sum_max;
  };
  second_stage(L.part_wout, g.w_out, (int64_t)Hkv * CL, col_chunks);
  second_stage(L.part_bout, g.b_out, Hkv, col_chunks);
  for (int l = 0; l < nl; ++l) second_stage(L.part_b[l], g.bias[l], (int64_t)Hkv * cnn.c_out[l], col_chunks);
  // 3. layers in reverse
  int cur = 0;
  for (int l = nl - 1; l >= 0; --l) {
    const int Cout = cnn.c_out[l], Cin = cin_of(l), ks = cnn.kernel[l];
    const float* dpre = L.dpre[cur];
    const WeightPlan W = weight_plan(cfg, cnn, l, total);
    const int64_t n_work = (int64_t)W.tiles * Hkv * W.groups * W.chunks;
    if (n_work > (int64_t)1 << 30) return hipErrorInvalidValue;
    const dim3 wgrid((unsigned)((n_work + 7) / 8 * 8));
    bool weights_done = false;
    if constexpr (kBf16) {
      if (W.split) {
        auto launch = [&](auto kernel, auto x0, auto x1, int at, int64_t st, int64_t sh) {
          hipLaunchKernelGGL(kernel, wgrid, dim3(256), 0, stream, x0, x1, at, st, sh, dpre, Cin, Cout, ks, cnn.dilation[l], L.seq_lo,
                             L.seq_hi, total, Hkv, W.tiles_n, W.tiles, W.groups, (int)n_work, W.chunk, L.part_w[l]);
        };
        if (l == 0) {
          const bf16_t *kp = static_cast<const bf16_t*>(k), *vp = static_cast<const bf16_t*>(v);
          if (W.wc == 2) launch(weight_split_kernel<bf16_t, 2, 2>, kp, vp, D, stride_tok, stride_head);
          else launch(weight_split_kernel<bf16_t, 1, 4>, kp, vp, D, stride_tok, stride_head);
        } else {
          auto kernel = W.wc == 2 ? (W.wm == 2 ? weight_split_kernel<float, 2, 2> : weight_split_kernel<float, 2, 1>)
                                  : (W.wm == 2 ? weight_split_kernel<float, 1, 2> : weight_split_kernel<float, 1, 1>);
          launch(kernel, in_of(l), in_of(l), Cin, (int64_t)Cin, total * Cin);
        }
        weights_done = true;
      }
    }
    if (!weights_done) {
      auto weight_product = W.wc == 2 ? (W.wm == 2 ? weight_product_kernel<2, 2> : weight_product_kernel<2, 1>)
                                      : (W.wm == 2 ? weight_product_kernel<1, 2> : weight_product_kernel<1, 1>);
      hipLaunchKernelGGL(weight_product, wgrid, dim3(256), 0, stream, in_of(l), dpre, Cin, Cout, ks, cnn.dilation[l], L.seq_lo,
                         L.seq_hi, total, Hkv, W.tiles_n, W.tiles, (int)n_work, W.chunk, L.part_w[l]);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    second_stage(L.part_w[l], g.w[l], (int64_t)Cout * Cin * ks * Hkv, W.chunks, ks, (int64_t)Cout * Cin);
    if (l > 0 || dk != nullptr || dv != nullptr) {
      // towards the input: contraction over this layer's output channels, taps mirrored
      bool done = false;
      if constexpr (std::is_same<T, bf16_t>::value) {
        if (on_bf16(l)) {   // bf16 weights, d y split into three bf16 terms
          const dim3 grid(tok_tiles, (unsigned)((Cin + TN - 1) / TN), (unsigned)Hkv);
          hipLaunchKernelGGL(Cin <= 32 ? conv_split_bf16_kernel<true> : conv_split_bf16_kernel<false>, grid, dim3(256), 0, stream,
                             dpre, static_cast<const bf16_t*>(L.wqf[l]), Cout, Cin, ks, cnn.dilation[l], -1, L.seq_lo, L.seq_hi,
                             total, Hkv, l > 0 ? 1 : 2, static_cast<const float*>(nullptr),
                             l > 0 ? L.pre[l - 1] : static_cast<const float*>(nullptr), L.dpre[cur ^ 1], static_cast<float*>(nullptr),
                             static_cast<bf16_t*>(dk), static_cast<bf16_t*>(dv), D, OutProj<bf16_t>{},
                             l > 0 ? L.part_b[l - 1] : static_cast<float*>(nullptr));
          if ((e = hipGetLastError()) != hipSuccess) return e;
          done = true;
        }
      }
      if (!done) {
      hipLaunchKernelGGL(conv_product(Cout, Cin), dim3(tok_tiles, (unsigned)((Cin + TN - 1) / TN), (unsigned)Hkv), dim3(256), 0,
                         stream, dpre, L.wb[l], Cout, Cin, ks, cnn.dilation[l], -1, L.seq_lo, L.seq_hi, total, Hkv,
                         l > 0 ? 1 : 2, static_cast<const float*>(nullptr),
                         l > 0 ? L.pre[l - 1] : static_cast<const float*>(nullptr), L.dpre[cur ^ 1],
                         static_cast<float*>(nullptr), static_cast<T*>(dk), static_cast<T*>(dv), D, OutProj<T>{},
                         l > 0 ? L.part_b[l - 1] : static_cast<float*>(nullptr));
      if ((e = hipGetLastError()) != hipSuccess) return e;
      }
    }
    cur ^= 1;
  }
  hipLaunchKernelGGL(chunk_sum_all_kernel, dim3((unsigned)((n_sum_max + 255) / 256), (unsigned)n_sums), dim3(256), 0, stream, sums);
  return hipGetLastError();
}

}  // namespace

size_t cnn_backward_workspace(const ltea_cfg& cfg, const ltea_cnn& cnn, int64_t total_tokens) {
  return carve(cfg, cnn, total_tokens, nullptr).bytes;
}
size_t cnn_backward_workspace_most(const ltea_cfg& cfg, const ltea_cnn& cnn, int64_t total_tokens) {
  return carve(cfg, cnn, total_tokens, nullptr, true).bytes;
}

hipError_t launch_cnn_backward(const ltea_cfg& cfg, const ltea_cnn& cnn, const void* k, const void* v,
                               int64_t stride_tok, int64_t stride_head, const SeqView& sv, const float* dz,
                               const ltea_cnn_grad& grad, void* dk, void* dv, void* workspace, hipStream_t stream) {
  if (sv.total_tokens == 0) {   // no tokens: every gradient is zero (a sum over no chunks)
    auto zero = [&](float* out, int64_t n) {
      hipLaunchKernelGGL(chunk_sum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                         static_cast<const float*>(nullptr), n, 0, out);
    };
    int cin = 2 * cfg.D;
    for (int l = 0; l < cnn.n_layers; ++l) {
      zero(grad.w[l], (int64_t)cfg.Hkv * cnn.c_out[l] * cin * cnn.kernel[l]);
      zero(grad.bias[l], (int64_t)cfg.Hkv * cnn.c_out[l]);
      cin = cnn.c_out[l];
    }
    zero(grad.w_out, (int64_t)cfg.Hkv * cin);
    zero(grad.b_out, cfg.Hkv);
    return hipGetLastError();
  }
  if (cfg.dtype == LTEA_F32)
    return run<float>(cfg, cnn, k, v, stride_tok, stride_head, sv, dz, grad, dk, dv, workspace, stream);
  return run<bf16_t>(cfg, cnn, k, v, stride_tok, stride_head, sv, dz, grad, dk, dv, workspace, stream);
}

}  // namespace ltea
