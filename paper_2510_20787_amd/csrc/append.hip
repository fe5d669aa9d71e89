// Continuation of a prefill onto an existing cache state (paper Section 3.1.3: the state after N tokens is the
// ring of the last w tokens plus the capped out-of-window segment; tokens dropped earlier are gone for good).
//
// Appending M new tokens to a sequence must give the rows and the final state of a one-shot prefill over all
// N + M tokens.  That holds because the kept set is nested: a token that is not among the top-b candidates of a
// prefix cannot be among the top-b of a longer one, so top-b over (old kept set + tokens leaving the window now)
// equals top-b over everything.
//
// The work is put in the shape the prefill kernels already handle.  Per sequence an "extended sequence" is laid out
// in the workspace:   [ pad | old kept entries ascending by position | ring tokens in position order | new tokens ]
// with the prefix (pad + kept entries) given the same length F for every head of the sequence, F >= budget chosen
// such that extended index and true position agree modulo the window (so that the ring slot of a token, position %
// window, can be computed from either).  Four launches:
//   1. the kernel of this file ranks the old kept entries, copies their rows, the ring's and the new ones into the
//      extended sequence and the keys that are already final (stored keys of the kept entries, ring logits below
//      n_old - rho) into its key array; pad rows are never read and stay unwritten;
//   2. the scoring kernel runs over the part whose logits are not final yet, packed on its own: the last
//      min(n_old, 2 rho) ring tokens and the new ones (a ring token below n_old - rho needs no new logit, one above it
//      has its whole left context in those rows);
//   3. the retention kernel runs over the extended sequence (candidates, top-b, gather, ring fill), taking each key
//      from the key array or from the fresh logits and writing kept positions back as true positions and, for the
//      attention kernel, in the ring + new frame (old kept entries get negative positions there and are visible
//      to every new query, as they should be); it also sets the counters;
//   4. the attention kernel runs with the ring + new part of the extended sequence as keys and the new tokens as
//      queries.
// Rotary models cache the keys after the rotation while the CNN scores them as they were before it.  For them the
// scoring rows are rotated back with the model's sinusoids (as in the batched scoring of the decode ring) where the
// caller does not pass the new tokens' unrotated keys.
#include "append_plan.h"
#include "ltea_common.h"
#include "ltea_kernels.h"
#include "rope_dev.h"

namespace ltea {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 128;      // items (kept entries, ring tokens, new tokens in this order) per workgroup
constexpr int kRankTile = 1024;  // positions compared against per LDS tile

struct BuildArgs {
  const char* k_new; const char* v_new; int64_t tok_bytes, head_bytes;   // new tokens [T][Hkv][D] view, in bytes
  const char* kf_new;                // the new tokens' keys as the CNN wants them (same view), or null
  const int32_t* cu_new;
  const char* k_win; const char* v_win; const float* win_score;
  const char* k_ret; const char* v_ret; const float* ret_score; const int32_t* ret_pos; const int32_t* ret_count;
  const int32_t* n_seen;
  char* k_ext; char* v_ext;          // [total_ext][Hkv][D] contiguous
  char* k_score; char* v_score;      // [total_score][Hkv][D] contiguous
  RopeDev rope;                      // cos == null: no rotation to undo
  int32_t* status;
  int n_seqs, Hkv, window, budget, rho, row_bytes;
};

// Grid (sequence x KV head, chunks of kItems items).  Bound: launch latency and the copies (at most budget + window + M
// rows of a head).  Every workgroup works its sequence's plan out itself (a sum over the sequences before it) and ranks
// only its own kept entries, 128 of them against all positions from LDS: as a launch of its own, with the positions
// read from memory one by one, the ranking of 512 entries took 39 us; with a trip to LDS per four of them a call of 4 x 384 tokens
// takes 59.4 us instead of 57.
template <typename T>
__global__ void __launch_bounds__(kThreads)
append_build_kernel(AppendPlan P, BuildArgs a) {
  constexpr int EPP = Elems<T>::N;
  __shared__ int sums[2][kThreads / kWave];
  __shared__ __align__(16) int pos_lds[kRankTile];
  __shared__ int rank_lds[kItems];
  const int b = blockIdx.x / a.Hkv, h = blockIdx.x - b * a.Hkv;
  const int64_t head = (int64_t)b * a.Hkv + h;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);

  // ---- plan: where this sequence's extended and scoring rows begin ----
  auto shape = [&](int s, int& N, int& wo, int& F, int& M) {
    N = a.n_seen[s];
    wo = N < a.window ? N : a.window;
    M = a.cu_new[s + 1] - a.cu_new[s];
    const int want = (N - wo) % a.window;                    // true position of the first ring token, modulo the window
    F = a.budget + ((want - a.budget) % a.window + a.window) % a.window;   // smallest F >= budget with F == want
  };
  int ext_before = 0, score_before = 0;
  for (int s = tid; s < b; s += kThreads) {
    int N, wo, F, M;
    shape(s, N, wo, F, M);
    ext_before += F + wo + M;
    score_before += min(wo, 2 * a.rho) + M;
  }
  ext_before = wave_sum_i(ext_before);
  score_before = wave_sum_i(score_before);
  if (lane == 0) { sums[0][tid / kWave] = ext_before; sums[1][tid / kWave] = score_before; }
  int N, wo, F, M;
  shape(b, N, wo, F, M);
  __syncthreads();
  const int e0 = sums[0][0] + sums[0][1] + sums[0][2] + sums[0][3];
  const int s0 = sums[1][0] + sums[1][1] + sums[1][2] + sums[1][3];
  const int ctx = min(wo, 2 * a.rho);                        // ring tokens in front of the scored new ones
  if (h == 0 && blockIdx.y == 0 && tid == 0) {
    P.n_old[b] = N; P.w_old[b] = wo; P.prefix[b] = F;
    P.cu_ext[b] = e0; P.cu_score[b] = s0;
    P.kv_start[b] = e0 + F; P.kv_len[b] = wo + M;
    if (b == a.n_seqs - 1) { P.cu_ext[b + 1] = e0 + F + wo + M; P.cu_score[b + 1] = s0 + ctx + M; }
  }

  const int cnt = a.budget > 0 ? a.ret_count[head] : 0, pad = F - cnt;
  if (blockIdx.y == 0 && tid == 0) P.old_count[head] = cnt;
  const int item0 = blockIdx.y * kItems, item_end = min(item0 + kItems, cnt + wo + M);
  if (item0 >= item_end) return;

  // ---- ranks of this workgroup's kept entries by position (positions are distinct): two threads per entry ----
  if (item0 < cnt) {                                         // uniform
    const int32_t* pos = a.ret_pos + head * a.budget;
    const int i = item0 + tid / 2;
    const int p = i < cnt ? pos[i] : 0;
    int rank = 0;
    for (int base = 0; base < cnt; base += kRankTile) {
      if (base > 0) __syncthreads();
#pragma unroll
      for (int u = 0; u < kRankTile / kThreads; ++u) {
        const int j = base + u * kThreads + tid;
        pos_lds[u * kThreads + tid] = j < cnt ? pos[j] : 0x7FFFFFFF;
      }
      __syncthreads();
      // eight quads requested before the first is used (those past the last entry hold 2^31 - 1): one by one each waits for its
      // trip to LDS
      const int quads = (min(cnt - base, kRankTile) + 3) / 4;
      for (int j = 0; j < quads; j += 16) {
        int4 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = reinterpret_cast<const int4*>(pos_lds)[j + 2 * u + (tid & 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) rank += (x[u].x < p) + (x[u].y < p) + (x[u].z < p) + (x[u].w < p);
      }
    }
    rank += __shfl_xor(rank, 1, kWave);
    if ((tid & 1) == 0 && i < cnt) {
      rank_lds[tid / 2] = rank;
      P.sorted_pos[head * a.budget + rank] = p;
      P.ext_key[(int64_t)h * P.total_ext + e0 + pad + rank] = a.ret_score[head * a.budget + i];
    }
    __syncthreads();
  }

  // ---- rows ----
  const int pieces = a.row_bytes / 16, rows_per_pass = kThreads / pieces;
  const int sub = tid / pieces, pc = tid - sub * pieces;
  const int64_t new0 = a.cu_new[b];
  bool out_of_tables = false;
  for (int item = item0 + sub; item < item_end; item += rows_per_pass) {
    const char *sk, *sv;
    int e;                      // extended index
    int sr = -1;                // scoring row
    int p_rot = -1;             // position whose rotation has to be undone for the scoring key
    const char* sf = nullptr;   // a row of ready-made scoring keys
    if (item < cnt) {
      e = pad + rank_lds[item - item0];
      sk = a.k_ret + (head * a.budget + item) * a.row_bytes;
      sv = a.v_ret + (head * a.budget + item) * a.row_bytes;
    } else if (item < cnt + wo) {
      const int r = item - cnt, p = N - wo + r;             // true position of this ring token
      const int slot = p % a.window;
      e = F + r;
      sk = a.k_win + (head * a.window + slot) * a.row_bytes;
      sv = a.v_win + (head * a.window + slot) * a.row_bytes;
      if (r >= wo - ctx) { sr = s0 + r - (wo - ctx); p_rot = p; }
      if (a.rope.cos != nullptr && p >= a.rope.n_pos) out_of_tables = true;
      if (pc == 0 && p < N - a.rho)                          // final before this call
        P.ext_key[(int64_t)h * P.total_ext + e0 + e] = a.win_score[head * a.window + slot];
    } else {
      const int r = item - cnt - wo;
      const int64_t t = new0 + r;
      e = F + wo + r;
      sk = a.k_new + t * a.tok_bytes + h * a.head_bytes;
      sv = a.v_new + t * a.tok_bytes + h * a.head_bytes;
      sr = s0 + ctx + r;
      if (a.kf_new != nullptr) sf = a.kf_new + t * a.tok_bytes + h * a.head_bytes;
      else p_rot = N + r;
    }
    const u32x4 xk = reinterpret_cast<const u32x4*>(sk)[pc];
    const u32x4 xv = reinterpret_cast<const u32x4*>(sv)[pc];
    const int64_t dst = ((int64_t)(e0 + e) * a.Hkv + h) * a.row_bytes;
    reinterpret_cast<u32x4*>(a.k_ext + dst)[pc] = xk;
    reinterpret_cast<u32x4*>(a.v_ext + dst)[pc] = xv;
    if (sr >= 0) {
      u32x4 xf = xk;
      if (sf != nullptr) {
        xf = reinterpret_cast<const u32x4*>(sf)[pc];
      } else if (a.rope.cos != nullptr && pc * EPP < a.rope.rot_dim) {
        if (p_rot >= a.rope.n_pos) out_of_tables = true;
        else xf = unrotate_piece<T>(a.rope, p_rot, pc * EPP, xk, reinterpret_cast<const T*>(sk));
      }
      const int64_t sdst = ((int64_t)sr * a.Hkv + h) * a.row_bytes;
      reinterpret_cast<u32x4*>(a.k_score + sdst)[pc] = xf;
      reinterpret_cast<u32x4*>(a.v_score + sdst)[pc] = xv;
    }
  }
  if (out_of_tables && a.status != nullptr) atomicOr(a.status, LTEA_ROPE_RANGE);
}

size_t up256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

// Upper bounds of the extended tokens and of the scored ones of all sequences (the true totals depend on device-side
// state).
int64_t append_ext_tokens(const ltea_cfg& cfg, int n_seqs, int64_t total_new) {
  return (int64_t)n_seqs * ((int64_t)cfg.budget + 2 * (int64_t)cfg.window) + total_new;
}
int64_t append_score_tokens(int n_seqs, int64_t total_new, int rho) { return total_new + (int64_t)n_seqs * 2 * rho; }

namespace {

struct Carved { AppendPlan plan; char *ext_k, *ext_v, *score_k, *score_v; float* score_logits; };

// Carves the workspace (integer arithmetic: a size query carves from a null base); returns the bytes used.
size_t carve(const ltea_cfg& cfg, int n_seqs, int64_t total_new, int rho, void* ws, Carved& c) {
  const int64_t ext = append_ext_tokens(cfg, n_seqs, total_new), scored = append_score_tokens(n_seqs, total_new, rho);
  const size_t esz = cfg.dtype == LTEA_F32 ? 4 : 2;
  uintptr_t p = reinterpret_cast<uintptr_t>(ws);
  auto take = [&](size_t bytes) { char* r = reinterpret_cast<char*>(p); p += up256(bytes); return r; };
  const size_t per_seq = sizeof(int32_t) * ((size_t)n_seqs + 1);
  AppendPlan& P = c.plan;
  P.n_old = reinterpret_cast<int32_t*>(take(per_seq));
  P.w_old = reinterpret_cast<int32_t*>(take(per_seq));
  P.prefix = reinterpret_cast<int32_t*>(take(per_seq));
  P.cu_ext = reinterpret_cast<int32_t*>(take(per_seq));
  P.cu_score = reinterpret_cast<int32_t*>(take(per_seq));
  P.kv_start = reinterpret_cast<int32_t*>(take(per_seq));
  P.kv_len = reinterpret_cast<int32_t*>(take(per_seq));
  const size_t per_entry = sizeof(int32_t) * (size_t)n_seqs * cfg.Hkv * (size_t)(cfg.budget > 0 ? cfg.budget : 1);
  P.old_count = reinterpret_cast<int32_t*>(take(sizeof(int32_t) * (size_t)n_seqs * cfg.Hkv));
  P.sorted_pos = reinterpret_cast<int32_t*>(take(per_entry));
  P.local_pos = reinterpret_cast<int32_t*>(take(per_entry));
  P.ext_key = reinterpret_cast<float*>(take((size_t)ext * cfg.Hkv * sizeof(float)));
  P.total_ext = ext;
  c.ext_k = take((size_t)ext * cfg.Hkv * cfg.D * esz);
  c.ext_v = take((size_t)ext * cfg.Hkv * cfg.D * esz);
  c.score_k = take((size_t)scored * cfg.Hkv * cfg.D * esz);
  c.score_v = take((size_t)scored * cfg.Hkv * cfg.D * esz);
  c.score_logits = reinterpret_cast<float*>(take((size_t)scored * cfg.Hkv * sizeof(float)));
  return (size_t)(p - reinterpret_cast<uintptr_t>(ws));
}

}  // namespace

size_t append_workspace(const ltea_cfg& cfg, int n_seqs, int64_t total_new, int rho) {
  Carved c;
  return carve(cfg, n_seqs, total_new, rho, nullptr, c);
}

// Stage 1 of the continuation; fills the device arrays that the later stages need.
hipError_t launch_append_build(const ltea_cfg& cfg, const void* k_new, const void* v_new, const void* kf_new,
                               int64_t stride_tok, int64_t stride_head, const int32_t* cu_new, int n_seqs,
                               int64_t total_new, int32_t max_new, int rho, const ltea_rope* rope, int32_t* status,
                               const ltea_cache& c, void* workspace, AppendBuffers* out, hipStream_t stream) {
  Carved w;
  carve(cfg, n_seqs, total_new, rho, workspace, w);
  const int64_t esz = cfg.dtype == LTEA_F32 ? 4 : 2;
  BuildArgs a;
  a.k_new = static_cast<const char*>(k_new); a.v_new = static_cast<const char*>(v_new);
  a.kf_new = static_cast<const char*>(kf_new);
  a.tok_bytes = stride_tok * esz; a.head_bytes = stride_head * esz; a.cu_new = cu_new;
  a.k_win = static_cast<const char*>(c.k_win); a.v_win = static_cast<const char*>(c.v_win); a.win_score = c.win_score;
  a.k_ret = static_cast<const char*>(c.k_ret); a.v_ret = static_cast<const char*>(c.v_ret);
  a.ret_score = c.ret_score; a.ret_pos = c.ret_pos; a.ret_count = c.ret_count; a.n_seen = c.n_seen;
  a.k_ext = w.ext_k; a.v_ext = w.ext_v; a.k_score = w.score_k; a.v_score = w.score_v;
  a.rope = rope_dev(rope); a.status = status;
  a.n_seqs = n_seqs; a.Hkv = cfg.Hkv; a.window = cfg.window; a.budget = cfg.budget; a.rho = rho;
  a.row_bytes = (int)(cfg.D * esz);
  const dim3 grid((unsigned)n_seqs * (unsigned)cfg.Hkv,
                  (unsigned)(((int64_t)cfg.budget + cfg.window + max_new + kItems - 1) / kItems));
  if (cfg.dtype == LTEA_F32) hipLaunchKernelGGL(append_build_kernel<float>, grid, dim3(kThreads), 0, stream, w.plan, a);
  else hipLaunchKernelGGL(append_build_kernel<bf16_t>, grid, dim3(kThreads), 0, stream, w.plan, a);
  out->plan = w.plan;
  out->ext_k = w.ext_k; out->ext_v = w.ext_v;
  out->score_k = w.score_k; out->score_v = w.score_v; out->score_logits = w.score_logits;
  out->total_score = append_score_tokens(n_seqs, total_new, rho);
  out->max_ext_len = cfg.budget + 2 * cfg.window + max_new;
  return hipGetLastError();
}

}  // namespace ltea
