// Scoring CNN of the LTE module (paper Section 3.1.1; Appendix A), generic layered path.
//
// Any depth, fp32 or bf16 storage, plain fp32 VALU arithmetic: one launch per conv layer (activations
// of layer l go through a [Hkv][T][C_l] fp32 scratch array), the last of which also forms the per-head output
// projection when its channels fit one workgroup.  It is the path for fp32 inputs and for bf16 shapes that the
// matrix-core kernels do not take.
#include <type_traits>

#include "ltea_common.h"
#include "ltea_kernels.h"

namespace ltea {
namespace {

constexpr int kTok = 16;       // tokens per workgroup
constexpr int kLanes = 16;     // output channels side by side; a thread owns CPT of them, 16 apart
constexpr int kChunk = 128;    // input channels per stage
constexpr int kStride = kChunk + 4;   // LDS row stride in floats: 16-byte reads of 16 rows at one column cover all banks

// 16 tokens x 16*CPT output channels of one KV head per workgroup, one (token, channel) sum per register.
// Input channels come through LDS in stages of 128 per tap (rows of the tap's positions, zeros outside the sequence, and
// the tap's weights), the next stage's loads in flight during this one's multiply-adds.  Every output is one chain
// bias, tap 0 channels 0.., tap 1 ... in this order.
// Bound: the latency of that chain (ks * Cin dependent multiply-adds, 640 for a k = 5 layer at D = 64, about 2 us) and of
// one trip to memory per stage; reading rows and weights from global memory inside the chain instead, one thread per
// output, took 77 us at 512 tokens x 2 heads (16 channels), this 9 us with the projection (was another launch of 4 us).
// act_in == null: input features are concat(K row, V row) of the token (2*D channels, keys first), else
// [Hkv][T][Cin] fp32.  Tap t reads position j + (t - (ks-1)/2) * dil of the same sequence; outside -> 0 (zero padding
// at every layer).  Output = Swish(bias + sum), to act_out; with logits given (last layer, all channels in this
// workgroup) the per-head projection b_out + sum_c w_out[c] * act[c] is formed here and only that is written.
template <typename T, int CPT>
__global__ void __launch_bounds__(kTok* kLanes)
conv_tile_kernel(const T* __restrict__ k, const T* __restrict__ v, int64_t stride_tok, int64_t stride_head, int D,
                 const float* __restrict__ act_in, const T* __restrict__ W, const float* __restrict__ bias, int Cin,
                 int Cout, int ks, int dil, const int32_t* __restrict__ cu, int n_seqs, int64_t total,
                 float* __restrict__ act_out, const T* __restrict__ w_out, const float* __restrict__ b_out,
                 float* __restrict__ logits) {
  constexpr int kThreads = kTok * kLanes;
  constexpr int kXPer = kTok * kChunk / kThreads, kWPer = CPT * kLanes * kChunk / kThreads;   // staged values per thread
  __shared__ __align__(16) float xs[kTok][kStride];
  __shared__ __align__(16) float ws[CPT * kLanes][kStride];
  __shared__ int64_t seq_lo[kTok], seq_hi[kTok];
  const int h = blockIdx.y, c0 = blockIdx.z * CPT * kLanes;
  const int64_t tok0 = (int64_t)blockIdx.x * kTok;
  const int tid = threadIdx.x, cl = tid % kLanes, tk = tid / kLanes;
  if (tid < kTok) {
    const int64_t tok = tok0 + tid < total ? tok0 + tid : total - 1;
    const int s = find_sequence(cu, n_seqs, tok);
    seq_lo[tid] = cu[s];
    seq_hi[tid] = cu[s + 1];
  }
  float acc[CPT];
#pragma unroll
  for (int i = 0; i < CPT; ++i) {
    const int c = c0 + cl + kLanes * i;
    acc[i] = c < Cout ? bias[(int64_t)h * Cout + c] : 0.f;
  }
  __syncthreads();

  // staging: thread owns column `col` of every (kThreads / kChunk)-th row
  const int col = tid % kChunk, row0 = tid / kChunk;
  constexpr int kRowStep = kThreads / kChunk;
  const int n_mc = (Cin + kChunk - 1) / kChunk, n_stages = ks * n_mc;
  float xr[kXPer], wr[kWPer];
  auto fetch = [&](int stage) {
    const int tap = stage / n_mc, m = (stage - tap * n_mc) * kChunk + col;
    const int64_t shift = (int64_t)(tap - (ks - 1) / 2) * dil;
    const bool m_ok = m < Cin;
#pragma unroll
    for (int i = 0; i < kXPer; ++i) {
      const int r = row0 + kRowStep * i;
      const int64_t p = tok0 + r + shift;
      const bool ok = m_ok && tok0 + r < total && p >= seq_lo[r] && p < seq_hi[r];
      const int64_t pc = ok ? p : 0;
      const int mc = ok ? m : 0;
      float x;
      if (act_in == nullptr) {
        const T* row = (mc < D ? k : v) + pc * stride_tok + (int64_t)h * stride_head;
        x = to_f32(row[mc < D ? mc : mc - D]);
      } else {
        x = act_in[((int64_t)h * total + pc) * Cin + mc];
      }
      xr[i] = ok ? x : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kWPer; ++i) {
      const int c = c0 + row0 + kRowStep * i;
      const bool ok = m_ok && c < Cout;
      const float w = to_f32(W[(((int64_t)h * Cout + (ok ? c : 0)) * Cin + (ok ? m : 0)) * ks + tap]);
      wr[i] = ok ? w : 0.f;
    }
  };
  fetch(0);
  for (int stage = 0; stage < n_stages; ++stage) {
    if (stage > 0) __syncthreads();   // everyone is done with the previous stage's rows
#pragma unroll
    for (int i = 0; i < kXPer; ++i) xs[row0 + kRowStep * i][col] = xr[i];
#pragma unroll
    for (int i = 0; i < kWPer; ++i) ws[row0 + kRowStep * i][col] = wr[i];
    __syncthreads();
    if (stage + 1 < n_stages) fetch(stage + 1);
#pragma unroll 4
    for (int m = 0; m < kChunk; m += 4) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(&xs[tk][m]);
#pragma unroll
      for (int i = 0; i < CPT; ++i) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(&ws[cl + kLanes * i][m]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i] = fmaf(x[e], w[e], acc[i]);
      }
    }
  }

  const int64_t tok = tok0 + tk;
  if (logits == nullptr) {
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = c0 + cl + kLanes * i;
      if (c < Cout && tok < total) act_out[((int64_t)h * total + tok) * Cout + c] = silu_f32(acc[i]);
    }
    return;
  }
  __syncthreads();                    // xs is free: it takes the activations and, after them, w_out
  float* wo = &ws[0][0];
#pragma unroll
  for (int i = 0; i < CPT; ++i) xs[tk][cl + kLanes * i] = silu_f32(acc[i]);
  if (tid < Cout) wo[tid] = to_f32(w_out[(int64_t)h * Cout + tid]);
  __syncthreads();
  if (tid < kTok && tok0 + tid < total) {
    float z = b_out[h];
    for (int c = 0; c < Cout; ++c) z = fmaf(xs[tid][c], wo[c], z);
    logits[(int64_t)h * total + tok0 + tid] = z;
  }
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

template <typename T>
hipError_t run(const ltea_cfg& cfg, const ltea_cnn& cnn, const void* k, const void* v, int64_t stride_tok,
               int64_t stride_head, const SeqView& sv, float* logits, void* workspace, hipStream_t stream) {
  const int64_t total = sv.total_tokens;
  int cmax = 0;
  for (int l = 0; l < cnn.n_layers; ++l) cmax = cnn.c_out[l] > cmax ? cnn.c_out[l] : cmax;
  float* buf[2] = {static_cast<float*>(workspace), static_cast<float*>(workspace) + (int64_t)cfg.Hkv * total * cmax};
  int cin = 2 * cfg.D;
  const float* act_in = nullptr;
  for (int l = 0; l < cnn.n_layers; ++l) {
    const int cout = cnn.c_out[l];
    float* act_out = buf[l & 1];
    // up to 64 channels fit one workgroup, which then also forms the projection of the last layer
    const int cpt = cout <= 16 ? 1 : cout <= 32 ? 2 : 4;
    const bool fused = l == cnn.n_layers - 1 && cout <= 16 * cpt;
    const dim3 tiles((unsigned)((total + kTok - 1) / kTok), (unsigned)cfg.Hkv, (unsigned)((cout + 16 * cpt - 1) / (16 * cpt)));
    auto go = [&](auto n) {
      hipLaunchKernelGGL((conv_tile_kernel<T, decltype(n)::value>), tiles, dim3(kTok * kLanes), 0, stream,
                         static_cast<const T*>(k), static_cast<const T*>(v), stride_tok, stride_head, cfg.D, act_in,
                         static_cast<const T*>(cnn.w[l]), cnn.bias[l], cin, cout, cnn.kernel[l], cnn.dilation[l],
                         sv.cu_seqlens, sv.n_seqs, total, act_out, static_cast<const T*>(cnn.w_out), cnn.b_out,
                         fused ? logits : nullptr);
    };
    if (cpt == 1) go(std::integral_constant<int, 1>{});
    else if (cpt == 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 4>{});
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
  int cmax = 0;
  for (int l = 0; l < cnn.n_layers; ++l) cmax = cnn.c_out[l] > cmax ? cnn.c_out[l] : cmax;
  const size_t one = (size_t)cfg.Hkv * (size_t)total_tokens * (size_t)cmax * sizeof(float);
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
