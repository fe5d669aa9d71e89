// Scoring CNN of the LTE module (paper Section 3.1.1; Appendix A), generic layered path.
//
// Any depth, fp32 or bf16 storage, fp32 arithmetic: one launch per conv layer (activations
// of layer l go through a [Hkv][T][C_l] fp32 scratch array), the last of which also forms the per-head output
// projection when its channels fit one workgroup.  It is the path for fp32 inputs and for bf16 shapes that the
// matrix-core kernels do not take.
#include <type_traits>

#include "ltea_common.h"
#include "ltea_kernels.h"

namespace ltea {
namespace {

constexpr int kTok = 16;       // tokens per workgroup
constexpr int kRun = 8;        // consecutive input channels per lane and step
constexpr int kWaves = 4;

// kRun consecutive elements as fp32; vec: 16-byte aligned and all there, else element by element up to `left`
__device__ __forceinline__ void load_run(const float* p, bool vec, int left, float (&x)[kRun]) {
  if (vec) {
    const f32x4 a = reinterpret_cast<const f32x4*>(p)[0], b = reinterpret_cast<const f32x4*>(p)[1];
#pragma unroll
    for (int e = 0; e < 4; ++e) { x[e] = a[e]; x[4 + e] = b[e]; }
  } else {
#pragma unroll
    for (int e = 0; e < kRun; ++e) x[e] = e < left ? p[e] : 0.f;
  }
}
__device__ __forceinline__ void load_run(const bf16_t* p, bool vec, int left, float (&x)[kRun]) {
  if (vec) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int e = 0; e < kRun; ++e) x[e] = to_f32(a[e]);
  } else {
#pragma unroll
    for (int e = 0; e < kRun; ++e) x[e] = e < left ? to_f32(p[e]) : 0.f;
  }
}

// 16 tokens x 16*NB output channels of one KV head per workgroup on v_mfma_f32_16x16x4_f32 (exact fp32 multiply-adds).
// The contraction over (input channel, tap) is dealt out in runs of 8 channels: run 16*step + 4*wave + lane group, every
// tap of it, so that a lane's weights are one contiguous piece of its channel's row ([channel][tap] order) and its token
// operand 8 consecutive values per tap row (zeros outside the sequence).  A layer of 128 input channels is one step: all
// operands are in flight together, and the four waves' partial sums meet once in LDS.
// Bound: latency (one trip to memory, 8*ks matrix instructions per wave).  512 tokens x 2 heads, k = 5, 128 -> 16
// channels: 77 us with one thread per output reading both operands from memory inside its chain, 18.7 us staged through
// LDS tap by tap, 6.4 us in this form (projection included, a launch of 4 us before).
// KS: kernel size compiled in (1, 3, 5, 7), 0: any.
// act_in == null: input features are concat(K row, V row) of the token (2*D channels, keys first), else
// [Hkv][T][Cin] fp32.  Tap t reads position j + (t - (ks-1)/2) * dil of the same sequence; outside -> 0 (zero padding
// at every layer).  Output = Swish(bias + sum), to act_out; with logits given (last layer, all channels in this
// workgroup) the per-head projection b_out + sum_c w_out[c] * act[c] is formed here and only that is written.
template <typename T, int NB, int KS>
__global__ void __launch_bounds__(kWaves* kWave)
conv_tile_kernel(const T* __restrict__ k, const T* __restrict__ v, int64_t stride_tok, int64_t stride_head, int D,
                 const float* __restrict__ act_in, const T* __restrict__ W, const float* __restrict__ bias, int Cin,
                 int Cout, int ks_any, int dil, const int32_t* __restrict__ cu, int n_seqs, int64_t total,
                 float* __restrict__ act_out, const T* __restrict__ w_out, const float* __restrict__ b_out,
                 float* __restrict__ logits) {
  const int ks = KS > 0 ? KS : ks_any;
  constexpr int kCh = 16 * NB, kPad = kCh + 1;
  __shared__ float part[kWaves][kTok][kPad];
  const int h = blockIdx.y, c0 = blockIdx.z * kCh;
  const int64_t tok0 = (int64_t)blockIdx.x * kTok;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int col = lane & 15, g = lane >> 4;       // operand row (token of A, channel of B) and lane group
  // weights in 16-byte pieces: every run full, rows and base aligned
  const bool w_vec = Cin % kRun == 0 && (reinterpret_cast<uintptr_t>(W) & 15u) == 0;
  const bool x_vec = act_in == nullptr || Cin % kRun == 0;

  f32x4 acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int64_t tok = tok0 + col < total ? tok0 + col : total - 1;
  int64_t lo = -1, hi = -1;                       // looked up under the weights' flight
  const int n_steps = (Cin + kRun * 4 * kWaves - 1) / (kRun * 4 * kWaves);
#pragma unroll 1
  for (int step = 0; step < n_steps; ++step) {
    const int m = kRun * (4 * (kWaves * step + wave) + g);
    const int left = Cin - m;                     // input channels from m on (<= 0: nothing to add)
    const int mc = left > 0 ? m : 0;
    auto weight_row = [&](int nb) {
      const int c = c0 + 16 * nb + col;
      return W + (((int64_t)h * Cout + (c < Cout ? c : 0)) * Cin + mc) * ks;
    };
    float w[NB][KS > 0 ? kRun * KS : 1];
    if constexpr (KS > 0) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int i = 0; i < KS; ++i) {
          float y[kRun];
          load_run(weight_row(nb) + kRun * i, w_vec, left * KS - kRun * i, y);
#pragma unroll
          for (int e = 0; e < kRun; ++e) w[nb][kRun * i + e] = y[e];
        }
    }
    if (lo < 0) {
      const int s = find_sequence(cu, n_seqs, tok);
      lo = cu[s];
      hi = cu[s + 1];
    }
    auto token_run = [&](int tap, float (&x)[kRun]) {
      const int64_t p = tok + (int64_t)(tap - (ks - 1) / 2) * dil;
      const bool ok = left > 0 && p >= lo && p < hi;
      const int64_t pc = ok ? p : tok;
      if (act_in == nullptr)
        load_run((mc < D ? k + mc : v + (mc - D)) + pc * stride_tok + (int64_t)h * stride_head, true, kRun, x);
      else
        load_run(act_in + ((int64_t)h * total + pc) * Cin + mc, x_vec, left, x);
#pragma unroll
      for (int e = 0; e < kRun; ++e) x[e] = ok ? x[e] : 0.f;
    };
    if constexpr (KS > 0) {
      float x[KS][kRun];
#pragma unroll
      for (int tap = 0; tap < KS; ++tap) token_run(tap, x[tap]);
#pragma unroll
      for (int tap = 0; tap < KS; ++tap)
#pragma unroll
        for (int e = 0; e < kRun; ++e)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[tap][e], w[nb][e * KS + tap], acc[nb], 0, 0, 0);
    } else {
      for (int tap = 0; tap < ks; ++tap) {
        float x[kRun];
        token_run(tap, x);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int e = 0; e < kRun; ++e) {
            const float wv = e < left ? to_f32(weight_row(nb)[e * ks + tap]) : 0.f;
            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], wv, acc[nb], 0, 0, 0);
          }
      }
    }
  }
  // register r of acc[nb] is token 4*g + r, channel 16*nb + col
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][4 * g + r][16 * nb + col] = acc[nb][r];
  __syncthreads();
  for (int i = tid; i < kTok * kCh; i += kWaves * kWave) {
    const int t = i / kCh, cc = i - t * kCh, c = c0 + cc;
    float y = 0.f;
    if (c < Cout) {
      y = bias[(int64_t)h * Cout + c];
#pragma unroll
      for (int w4 = 0; w4 < kWaves; ++w4) y += part[w4][t][cc];
      y = silu_f32(y);
      if (logits == nullptr && tok0 + t < total) act_out[((int64_t)h * total + tok0 + t) * Cout + c] = y;
    }
    part[0][t][cc] = y;      // read above by this thread only
  }
  if (logits == nullptr) return;
  __syncthreads();
  // 16 lanes per token, channels 16 apart, fixed order
  const int t = tid / 16;
  float z = 0.f;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int c = 16 * nb + tid % 16;
    if (c < Cout) z = fmaf(part[0][t][c], to_f32(w_out[(int64_t)h * Cout + c]), z);
  }
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) z += __shfl_xor(z, off, kWave);
  if (tid % 16 == 0 && tok0 + t < total) logits[(int64_t)h * total + tok0 + t] = z + b_out[h];
}

// logits[h][t] = b_out[h] + sum_c w_out[h][c] * act[h][t][c]  (last layers too wide for one workgroup)
template <typename T>
__global__ void __launch_bounds__(256)
out_proj_kernel(const float* __restrict__ act, const T* __restrict__ w_out, const float* __restrict__ b_out, int C,
                int64_t total, float* __restrict__ logits) {
  const int h = blockIdx.y;
  const int64_t tok = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tok >= total) return;
  const float* a = act + ((int64_t)h * total + tok) * C;
  float acc = b_out[h];
  for (int c = 0; c < C; ++c) acc = fmaf(a[c], to_f32(w_out[(int64_t)h * C + c]), acc);
  logits[(int64_t)h * total + tok] = acc;
}

// Floats of one activation array, in whole 256-byte pieces: rows of a multiple of kRun channels then start on 16-byte
// boundaries in both arrays, as the vector loads of the next layer assume.
size_t activation_floats(const ltea_cfg& cfg, const ltea_cnn& cnn, int64_t total) {
  int cmax = 0;
  for (int l = 0; l < cnn.n_layers; ++l) cmax = cnn.c_out[l] > cmax ? cnn.c_out[l] : cmax;
  return ((size_t)cfg.Hkv * (size_t)total * (size_t)cmax + 63) / 64 * 64;
}

template <typename T>
hipError_t run(const ltea_cfg& cfg, const ltea_cnn& cnn, const void* k, const void* v, int64_t stride_tok,
               int64_t stride_head, const SeqView& sv, float* logits, void* workspace, hipStream_t stream) {
  const int64_t total = sv.total_tokens;
  float* buf[2] = {static_cast<float*>(workspace), static_cast<float*>(workspace) + activation_floats(cfg, cnn, total)};
  int cin = 2 * cfg.D;
  const float* act_in = nullptr;
  for (int l = 0; l < cnn.n_layers; ++l) {
    const int cout = cnn.c_out[l];
    float* act_out = buf[l & 1];
    // up to 64 channels fit one workgroup, which then also forms the projection of the last layer
    const int cpt = cout <= 16 ? 1 : cout <= 32 ? 2 : 4;
    const bool fused = l == cnn.n_layers - 1 && cout <= 16 * cpt;
    const dim3 tiles((unsigned)((total + kTok - 1) / kTok), (unsigned)cfg.Hkv, (unsigned)((cout + 16 * cpt - 1) / (16 * cpt)));
    auto go = [&](auto nb, auto k_size) {
      hipLaunchKernelGGL((conv_tile_kernel<T, decltype(nb)::value, decltype(k_size)::value>), tiles, dim3(kWaves * kWave),
                         0, stream, static_cast<const T*>(k), static_cast<const T*>(v), stride_tok, stride_head, cfg.D,
                         act_in, static_cast<const T*>(cnn.w[l]), cnn.bias[l], cin, cout, cnn.kernel[l], cnn.dilation[l],
                         sv.cu_seqlens, sv.n_seqs, total, act_out, static_cast<const T*>(cnn.w_out), cnn.b_out,
                         fused ? logits : nullptr);
    };
    auto by_width = [&](auto k_size) {
      if (cpt == 1) go(std::integral_constant<int, 1>{}, k_size);
      else if (cpt == 2) go(std::integral_constant<int, 2>{}, k_size);
      else go(std::integral_constant<int, 4>{}, k_size);
    };
    switch (cnn.kernel[l]) {
      case 1: by_width(std::integral_constant<int, 1>{}); break;
      case 3: by_width(std::integral_constant<int, 3>{}); break;
      case 5: by_width(std::integral_constant<int, 5>{}); break;
      case 7: by_width(std::integral_constant<int, 7>{}); break;
      default: by_width(std::integral_constant<int, 0>{});
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || fused) return e;
    act_in = act_out;
    cin = cout;
  }
  dim3 grid((unsigned)((total + 255) / 256), (unsigned)cfg.Hkv);
  hipLaunchKernelGGL(out_proj_kernel<T>, grid, dim3(256), 0, stream, act_in, static_cast<const T*>(cnn.w_out),
                     cnn.b_out, cin, total, logits);
  return hipGetLastError();
}

}  // namespace

size_t score_generic_workspace(const ltea_cfg& cfg, const ltea_cnn& cnn, int64_t total_tokens) {
  const size_t one = activation_floats(cfg, cnn, total_tokens) * sizeof(float);
  return cnn.n_layers > 1 ? 2 * one : one;
}

hipError_t launch_score_generic(const ltea_cfg& cfg, const ltea_cnn& cnn, const void* k, const void* v,
                                int64_t stride_tok, int64_t stride_head, const SeqView& sv, float* logits,
                                void* workspace, hipStream_t stream) {
  if (sv.total_tokens == 0) return hipSuccess;
  if (cfg.dtype == LTEA_F32)
    return run<float>(cfg, cnn, k, v, stride_tok, stride_head, sv, logits, workspace, stream);
  return run<bf16_t>(cfg, cnn, k, v, stride_tok, stride_head, sv, logits, workspace, stream);
}

}  // namespace ltea
