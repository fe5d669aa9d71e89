// Launchers of the decode step and the packing of receptive-field windows for CNNs that are scored outside it.  The step
// itself is described in decode_step.h.
#include "decode_run.h"

namespace ltea {
namespace {

size_t up256(size_t x) { return (x + 255) / 256 * 256; }

// Receptive-field windows of the token being finalised, packed for the prefill scoring kernels (CNNs whose activation rows
// do not fit the step's LDS): sequence b gets rows b*R .. b*R + len - 1 (R = 2*rho + 1) holding positions
// max(0, t - 2*rho) .. t (the ring rows and, last, the incoming token); a second, possibly empty pseudo-sequence covers
// the unused rest of the R rows so that the packing stays contiguous without a prefix sum over the batch:
// cu2[2b] = b*R, cu2[2b+1] = b*R + len, cu2[2B] = B*R.
// Rotary models (rope.cos != null): the ring holds rotated keys, which are rotated back here; the incoming token's
// scoring key is kf_new when given, else k_new rotated back at position t.
// One workgroup of 256 threads per sequence b.
template <typename T>
__global__ void __launch_bounds__(256)
decode_windows_kernel(CacheDev C, const T* __restrict__ k_new, const T* __restrict__ v_new, const T* __restrict__ kf_new,
                      RopeDev rope, int32_t* __restrict__ status, T* __restrict__ win_k, T* __restrict__ win_v,
                      int32_t* __restrict__ cu2, int B, int Hkv, int D, int window, int rho) {
  constexpr int EPP = Elems<T>::N;
  const int b = blockIdx.x, R = 2 * rho + 1;
  const int t = C.n_seen[b];
  const int first = t - 2 * rho > 0 ? t - 2 * rho : 0;
  const int len = t - first + 1;
  const int pieces = D / EPP;                                 // 16-byte pieces per row
  if (threadIdx.x == 0) {
    cu2[2 * b] = b * R;
    cu2[2 * b + 1] = b * R + len;
    if (b == B - 1) cu2[2 * B] = B * R;
  }
  const int items = len * Hkv * pieces;
  bool out_of_tables = false;
  for (int i = threadIdx.x; i < items; i += 256) {
    const int pc = i % pieces, h = (i / pieces) % Hkv, r = i / (pieces * Hkv);
    const int p = first + r;
    const int64_t head = (int64_t)b * Hkv + h;
    const T* sk = p == t ? k_new + head * D : static_cast<const T*>(C.k_win) + (head * window + p % window) * D;
    const T* sv = p == t ? v_new + head * D : static_cast<const T*>(C.v_win) + (head * window + p % window) * D;
    const int64_t dst = ((int64_t)(b * R + r) * Hkv + h) * D;
    u32x4 xk = reinterpret_cast<const u32x4*>(sk)[pc];
    if (p == t && kf_new != nullptr) {
      xk = reinterpret_cast<const u32x4*>(kf_new + head * D)[pc];
    } else if (rope.cos != nullptr && pc * EPP < rope.rot_dim) {
      if (p >= rope.n_pos) out_of_tables = true;
      else xk = unrotate_piece<T>(rope, p, pc * EPP, xk, sk);
    }
    reinterpret_cast<u32x4*>(win_k + dst)[pc] = xk;
    reinterpret_cast<u32x4*>(win_v + dst)[pc] = reinterpret_cast<const u32x4*>(sv)[pc];
  }
  if (out_of_tables && status != nullptr) atomicOr(status, LTEA_ROPE_RANGE);
}

hipError_t launch_step(const ltea_cfg& cfg, const ltea_cnn* cnn_or_null, const StepInputs& in, const ltea_cache& c, int n_seqs,
                       void* workspace, hipStream_t stream, const float* given = nullptr, int64_t given_total = 0) {
  if (n_seqs == 0) return hipSuccess;
  if (cfg.dtype == LTEA_F32)
    return cfg.D == 64 ? decode_run_f32_64(cfg, cnn_or_null, in, c, n_seqs, workspace, given, given_total, stream)
                       : decode_run_f32_128(cfg, cnn_or_null, in, c, n_seqs, workspace, given, given_total, stream);
  return cfg.D == 64 ? decode_run_bf16_64(cfg, cnn_or_null, in, c, n_seqs, workspace, given, given_total, stream)
                     : decode_run_bf16_128(cfg, cnn_or_null, in, c, n_seqs, workspace, given, given_total, stream);
}

}  // namespace

// Shares of a head's rows (one workgroup each): one per 64 KB of rows as long as there is at most one workgroup per CU.
// A CU alone streams about 64 KB per us, handing shares over costs about 5 us: one share per 1 MB / 256 KB / 128 KB / 64 KB
// measured, in us per lazy step, 25 / 15.3 / 12.7 / 11.8 (one sequence of 16 heads x 1536 rows of D = 128), 46 / 16.9 / 16.1
// / 16.2 (32 heads x 3072 rows), 13.9 / 13.8 / 12.8 / 12.1 (8 heads x 1280 rows of D = 64); more workgroups than CUs gained
// nothing (16 sequences of the latter: 15.9 -> 18.1).  At least 128 rows per share: fp32 rows of D = 128 are 1 KB, and records for
// twice the shares would not fit the fixed scratch of ltea_decode_step_static where a group has 64 query heads and more.
namespace {
int64_t shares_by_rows(const ltea_cfg& cfg) {
  const int64_t rows = (int64_t)cfg.window + cfg.budget, bytes = rows * 2 * cfg.D * (cfg.dtype == LTEA_F32 ? 4 : 2);
  const int64_t by_bytes = bytes / (64 * 1024), by_rows = (rows + 127) / 128;
  const int64_t n = by_bytes < by_rows ? by_bytes : by_rows;
  return n < 1 ? 1 : n > 64 ? 64 : n;
}
size_t workspace_of(const ltea_cfg& cfg, int n_seqs, int64_t shares /* of all sequences, per KV head */) {
  return ((size_t)shares * cfg.Hq * (cfg.D + 2) + (size_t)n_seqs * cfg.Hkv) * sizeof(float) +
         ((size_t)n_seqs + (size_t)n_seqs * cfg.Hkv) * sizeof(int32_t);
}
}  // namespace

int decode_num_splits(const ltea_cfg& cfg, int n_seqs) {
  const int64_t heads = (int64_t)n_seqs * cfg.Hkv, n = shares_by_rows(cfg);
  const int64_t by_cus = heads > 0 ? 256 / heads : n;
  return by_cus < 1 ? 1 : (int)(n < by_cus ? n : by_cus);
}

size_t decode_workspace(const ltea_cfg& cfg, int n_seqs) {
  return workspace_of(cfg, n_seqs, (int64_t)n_seqs * decode_num_splits(cfg, n_seqs));
}

size_t decode_workspace_most(const ltea_cfg& cfg, int n_seqs) {
  const int64_t shared = n_seqs * shares_by_rows(cfg), by_cus = 256 / cfg.Hkv;
  const int64_t most = shared < by_cus ? shared : by_cus;
  return workspace_of(cfg, n_seqs, most > n_seqs ? most : n_seqs);
}

// The documented bound on the CNN, for two generations of activation rows of the whole receptive field (the launch keeps
// only every unit-th row of them in LDS, in whole quads, beside the step's own 69 KB at most).
bool decode_scores_inside(const ltea_cfg& cfg, const ltea_cnn& cnn) {
  return (size_t)2 * (2 * cnn_rho(&cnn) + 1) * widest_row(cfg, cnn) * sizeof(float) <= 48 * 1024;
}

hipError_t launch_decode_step(const ltea_cfg& cfg, const ltea_cnn& cnn, const ltea_rope* rope, const void* q, const void* k,
                              const void* v, const void* k_feat, void* out, const ltea_cache& c, int n_seqs,
                              int32_t* status, void* workspace, hipStream_t stream) {
  return launch_step(cfg, &cnn, StepInputs{q, k, v, k_feat, rope, out, status}, c, n_seqs, workspace, stream);
}

size_t decode_windows_layout(const ltea_cfg& cfg, int rho, int n_seqs, void* base, DecodeWindows* out) {
  const size_t esz = cfg.dtype == LTEA_F32 ? 4 : 2;
  const size_t rows = (size_t)n_seqs * (2 * rho + 1);
  uintptr_t p = reinterpret_cast<uintptr_t>(base);
  auto take = [&](size_t bytes) { char* r = reinterpret_cast<char*>(p); p += up256(bytes); return r; };
  void* wk = take(rows * cfg.Hkv * cfg.D * esz);
  void* wv = take(rows * cfg.Hkv * cfg.D * esz);
  int32_t* cu2 = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (2 * (size_t)n_seqs + 1)));
  float* lg = reinterpret_cast<float*>(take(sizeof(float) * rows * cfg.Hkv));
  if (out) { out->win_k = wk; out->win_v = wv; out->cu2 = cu2; out->logits = lg; out->total = (int64_t)rows; }
  return (size_t)(p - reinterpret_cast<uintptr_t>(base));
}

hipError_t launch_decode_windows(const ltea_cfg& cfg, int rho, const void* k, const void* v, const void* k_feat,
                                 const ltea_rope* rope, int32_t* status, const ltea_cache& c, int n_seqs,
                                 const DecodeWindows& w, hipStream_t stream) {
  CacheDev C{c.k_win, c.v_win, c.win_score, c.k_ret, c.v_ret, c.ret_score, c.ret_pos, c.ret_count, c.n_seen, c.n_scored};
  auto go = [&](auto tag) {
    using T = decltype(tag);
    hipLaunchKernelGGL(decode_windows_kernel<T>, dim3((unsigned)n_seqs), dim3(256), 0, stream, C,
                       static_cast<const T*>(k), static_cast<const T*>(v), static_cast<const T*>(k_feat), rope_dev(rope),
                       status, static_cast<T*>(w.win_k), static_cast<T*>(w.win_v), w.cu2, n_seqs, cfg.Hkv, cfg.D,
                       cfg.window, rho);
  };
  if (cfg.dtype == LTEA_F32) go(float{});
  else go(bf16_t{});
  return hipGetLastError();
}

hipError_t launch_decode_step_scored(const ltea_cfg& cfg, const ltea_cnn& cnn, const void* q, const void* k,
                                     const void* v, void* out, const ltea_cache& c, int n_seqs, void* workspace,
                                     const float* logits, int64_t logits_total, hipStream_t stream) {
  return launch_step(cfg, &cnn, StepInputs{q, k, v, nullptr, nullptr, out, nullptr}, c, n_seqs, workspace, stream, logits,
                     logits_total);
}

hipError_t launch_decode_step_lazy(const ltea_cfg& cfg, const void* q, const void* k, const void* v, void* out,
                                   const ltea_cache& c, int n_seqs, int32_t* status, void* workspace,
                                   hipStream_t stream) {
  return launch_step(cfg, nullptr, StepInputs{q, k, v, nullptr, nullptr, out, status}, c, n_seqs, workspace, stream);
}

}  // namespace ltea
